"""An orbital that the input check accepts, 8e-13 of its power outside the
declared band (tolerance 1e-12): float64 plans that check give the energy of the
caller's grid, to which such content is second order."""
import pytest
import torch

from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu

H = 23.5 / 96


@pytest.mark.parametrize("axis", [1, 2, 3])
@pytest.mark.parametrize("n", [64, 96])
def test_accepted_admixture_is_second_order(n, axis):
    n_orb = 9
    box = (n * H,) * 3
    psi = torch.from_numpy(generate.random_pw((n, n, n), box, n_orb, 5.0, 4)).cuda()
    # shifted by half the grid's frequencies along one axis: on every other point
    # this is psi itself, far outside the band everywhere else
    sign = 1.0 - 2.0 * (torch.arange(n, device="cuda", dtype=torch.float64) % 2)
    shape = [1, 1, 1, 1]
    shape[axis] = n
    leaky = psi * (1.0 + 0.9e-6 * sign.view(shape))
    spec = hfx.SystemSpec(n, box, n_orb)
    e = hfx.Plan(spec, hfx.FP64).exchange_energy(psi)
    plan = hfx.Plan(spec, hfx.FP64, "ecut=5;check=1")
    # second order: a few times 0.9e-6^2, and rounding
    assert float((plan.exchange_energy(leaky) - e).abs()) <= 1e-11 * float(e.abs())
    kpsi, ex = plan.apply_exchange(leaky)
    assert torch.equal(ex, plan.exchange_energy(leaky))
    with pytest.raises(hfx.HfxError, match="input check"):
        plan.exchange_energy(psi * (1.0 + 1.5e-6 * sign.view(shape)))
