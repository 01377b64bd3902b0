"""Several systems on reduced pair grids: streams of their own by default, shared
launches with group=1, the same results bit for bit."""
import pytest
import torch

from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu

H = 23.5 / 96


@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["f32", "f64"])
def test_reduced_systems_fork_by_default(prec):
    n, counts = 64, (20, 18, 20)
    box = (n * H,) * 3
    psi = torch.from_numpy(generate.random_pw((n,) * 3, box, sum(counts), 5.0, 2)).cuda().reshape(-1)
    specs = [hfx.SystemSpec(n, box, k) for k in counts]
    out = {}
    for group in ("", ";group=0", ";group=1"):
        plan = hfx.Plan(specs, prec, "ecut=5;variant=" + hfx.variants(n, prec)[0] + group)
        assert "->" in plan.describe(1)
        assert ("/3" in plan.describe(1).split("class=")[1]) == (group == ";group=1")
        out[group] = plan.apply_exchange(psi)
    for group in (";group=0", ";group=1"):
        assert torch.equal(out[""][0], out[group][0]) and torch.equal(out[""][1], out[group][1])
