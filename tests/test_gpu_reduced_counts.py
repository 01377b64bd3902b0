"""Where plans that leave the kernel configuration open take the reduced pair
grids: the band fits and the orbitals are enough.  On both sides of each line the
results are those of the caller's grid (the bars of the parity test of the reduced
grids), and so they are at every small count when the reduced grid is asked for
by name."""
import pytest
import torch

from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu

H = 23.5 / 96
LINES = {hfx.FP32: {64: 44, 72: 26, 80: 18, 96: 28, 108: 9, 120: 17, 128: 10},
         hfx.FP64: {64: 17, 72: 17, 80: 13, 96: 17, 108: 9, 120: 10, 128: 9}}


def _orbitals(n, box, n_orb):
    """Combinations of a few orbitals of the 5 Ha sphere."""
    few = torch.from_numpy(generate.random_pw((n,) * 3, box, 6, 5.0, 3)).cuda().view(6, -1)
    gen = torch.Generator(device="cuda").manual_seed(n_orb)
    mix = torch.randn(n_orb, 6, generator=gen, device="cuda", dtype=torch.float64)
    return (mix @ few).view(n_orb, n, n, n)


def _check(spec, prec, options, reduced, psi):
    plan = hfx.Plan(spec, prec, options)
    assert ("->" in plan.describe()) == reduced and "pair_grid=" in plan.describe()
    k0, e0 = hfx.Plan(spec, prec).apply_exchange(psi)
    k1, e1 = plan.apply_exchange(psi)
    k, e = (1e-10, 1e-12) if prec == hfx.FP64 else (2e-6, 2e-7)
    assert float((k1.double() - k0.double()).abs().max()) <= k * float(k0.abs().max())
    assert float((e1 - e0).abs().max()) <= e * float(e0.abs().max())
    return plan, k1


@pytest.mark.parametrize("n", [64, 72, 80, 96, 108, 120, 128])
@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["f32", "f64"])
def test_both_sides_of_the_line(n, prec):
    box = (n * H,) * 3
    for n_orb in (LINES[prec][n] - 1, LINES[prec][n]):
        psi = _orbitals(n, box, n_orb)
        _check(hfx.SystemSpec(n, box, n_orb), prec, "ecut=5", n_orb == LINES[prec][n], psi)


@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["f32", "f64"])
@pytest.mark.parametrize("n,box,n_orb", [
    (64, (64 * H,) * 3, 1), (64, (64 * H,) * 3, 8), (64, (64 * H,) * 3, 16), (64, (15.0, 12.0, 14.0), 5),
    (72, (72 * H,) * 3, 19), (96, (96 * H,) * 3, 9), (120, (120 * H,) * 3, 9)])
def test_small_sets_by_name(n, box, n_orb, prec):
    psi = _orbitals(n, box, n_orb)
    spec = hfx.SystemSpec(n, box, n_orb)
    plan, k = _check(spec, prec, "ecut=5;variant=" + hfx.variants(n, prec)[0], True, psi)
    g = torch.empty_like(k)
    graph = plan.graph(hfx.GRAPH_APPLY, psi, g)
    for _ in range(3):
        g.zero_()
        graph.launch()
        assert torch.equal(g, k)
