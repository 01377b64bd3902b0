"""Rows per tile pair of screened plans: 32 by default from 80^3 on (where the
batches hold such a tile pair), the caller's otherwise.  Against the same
screening on 8 rows: the same pairs, other sums' order.  float64 differs by
n 2^-53 of the sums (1e-13 at these sizes), float32 K psi by n 2^-24 (41 terms:
2.5e-6 of the largest); float32 energies add float32 pair sums in float64."""
import pytest
import torch

from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("n,n_orb,rows", [(72, 41, 16), (80, 41, 32), (80, 16, 16), (80, 33, 32),
                                          (96, 9, 16)])
def test_default_rows_of_screened_plans(n, n_orb, rows, prec):
    box = (n * 23.5 / 96,) * 3
    psi = torch.from_numpy(generate.gaussians((n,) * 3, box, n_orb, 20.0, 17)[0]).cuda()
    spec = hfx.SystemSpec(n, box, n_orb, hfx.ERFC, 0.106)
    plan, tall = hfx.Plan(spec, prec, "ecut=20"), hfx.Plan(spec, prec, "ecut=20;rows=8")
    before = plan.describe()
    kept = plan.screen(psi, 2e-2)
    assert 0 < kept[0] < n_orb * (n_orb + 1) // 2 and tall.screen(psi, 2e-2) == kept
    assert " rows=%d " % rows in plan.describe() and " rows=8 " in tall.describe()
    assert plan.schedule_info()[2:] == (tall.schedule_info()[2], kept[0])
    (k, e), (k8, e8) = plan.apply_exchange(psi), tall.apply_exchange(psi)
    bar = 1e-13 if prec == hfx.FP64 else n_orb * 2.0 ** -24
    assert float((k - k8).abs().max()) <= bar * float(k8.abs().max())
    assert abs(float((e - e8) / e8)) <= 1e-12
    k2 = plan.apply_exchange(psi)[0]
    assert torch.equal(k, k2)
    plan.screen(psi, 0.0)
    assert plan.describe() == before
