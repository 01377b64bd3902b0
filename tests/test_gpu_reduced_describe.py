"""What a plan on reduced pair grids reports: the schedules and threads of the
kernels that run, and the bytes and flops of the work done."""
import pytest
import torch

from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu

H = 23.5 / 96


def _product(schedule):
    p = 1
    for r in schedule.split("x"):
        p *= int(r)
    return p


@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["f32", "f64"])
@pytest.mark.parametrize("n,m", [(64, 48), (120, 96)])
def test_describe_and_tallies(n, m, prec):
    n_orb, elem = 9, 4 if prec == hfx.FP32 else 8
    box = (n * H,) * 3
    name = hfx.variants(n, prec)[0]
    plan = hfx.Plan(hfx.SystemSpec(n, box, n_orb), prec, "ecut=5;variant=" + name)
    d = dict(x.split("=", 1) for x in plan.describe().split())
    assert d["variant"] == name and d["n"] == str(n) and d["pair_grid"] == "%d->%d" % (n // 2, m)
    for axis in "xyz":
        forward, inverse = d[axis].split("/")
        assert _product(forward) == n // 2 and _product(inverse) == m
    assert d["plane"] == "fused" and d["y_rows"] == d["x_cols"] == "half"
    assert d["z_fwd"] == "half(" + d["z"].split("/")[0] + ")"
    psi = torch.from_numpy(generate.random_pw((n,) * 3, box, n_orb, 5.0, 2)).cuda()
    plan.profile(True)
    plan.apply_exchange(psi)
    r = plan.profile_read()
    assert r["zero"]["bytes"] == n_orb * m ** 3 * elem
    if prec == hfx.FP32:  # the pair means, on the samples
        assert r["contract"]["bytes"] == n_orb * (n // 2) ** 3 * 8
        assert r["contract"]["flops"] == 2 * n_orb ** 2 * (n // 2) ** 3
    there = n ** 3 * 8 + (n // 2) ** 3 * (12 if prec == hfx.FP32 else 8) + m ** 3 * elem
    back = (n ** 3 + m ** 3 * (2 if prec == hfx.FP32 else 1)) * elem
    assert r["stage"]["bytes"] == n_orb * (there + back)
