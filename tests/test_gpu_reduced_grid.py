"""Reduced pair grids (band-limited plans whose grid oversamples the pair
densities twofold): every exchange call against the same call on the caller's
full grid, which a plan without a declared cutoff runs.

Both paths are exact for such orbitals, so they differ by rounding alone.
float64: the bars of the parity tests against the oracle (1e-12 of E_x, 1e-10
of max |K psi|).  float32: twice the path's own error against float64, which
the parity tests bound by 1e-7 of E_x and which is below 1e-6 of max |K psi|
(2^-24 through six transforms of at most 128 points)."""
import numpy as np
import pytest
import torch

from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu

GRIDS = [(64, 64), (72, 72), (80, 80), (96, 96), (108, 108), (120, 120), (128, 128), (64, 128)]
H = 23.5 / 96


def _case(n, nz, n_orb, seed=3):
    box = (n * H, n * H, nz * H)
    psi = generate.random_pw((nz, n, n), box, n_orb, 5.0, seed)
    return box, torch.from_numpy(psi).cuda()


def _spec(n, nz, box, n_orb, kernel=hfx.TRUNCATED, param=0.0):
    return hfx.SystemSpec(n if n == nz else (n, n, nz), box, n_orb, kernel, param)


def _close(a, b, prec, energy=False):
    bar = (1e-12 if energy else 1e-10) if prec == hfx.FP64 else (2e-7 if energy else 2e-6)
    a, b = a.double(), b.double()
    assert float((a - b).abs().max()) <= bar * float(b.abs().max())


@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["f32", "f64"])
@pytest.mark.parametrize("n,nz", GRIDS)
def test_reduced_matches_full_grid(n, nz, prec):
    n_orb = 19 if n <= 80 else 9  # a full tile pair and a ragged one
    box, psi = _case(n, nz, n_orb)
    spec = _spec(n, nz, box, n_orb)
    full, red = hfx.Plan(spec, prec), hfx.Plan(spec, prec, "ecut=5")
    assert "pair_grid=" in red.describe() and "pair_grid=" not in full.describe()
    k0, e0 = full.apply_exchange(psi)
    k1, e1 = red.apply_exchange(psi)
    _close(k1, k0, prec)
    _close(e1, e0, prec, True)
    assert torch.equal(red.apply_exchange(psi)[0], k1)  # reproducible
    _close(red.exchange_energy(psi), e0, prec, True)
    _close(red.exchange_gradient(psi), 2 * spec.dv * k0.double(), prec)
    g = torch.empty_like(k1)
    graph = red.graph(hfx.GRAPH_APPLY, psi, g)
    for _ in range(3):
        g.zero_()
        graph.launch()
        assert torch.equal(g, k1)


@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["f32", "f64"])
@pytest.mark.parametrize("n_orb", [1, 8, 16, 37])
def test_orbital_counts_streams_and_shards(n_orb, prec):
    n = 64
    box, psi = _case(n, n, n_orb)
    spec = _spec(n, n, box, n_orb, hfx.ERFC, 0.106)
    k0, e0 = hfx.Plan(spec, prec).apply_exchange(psi)
    k1, e1 = hfx.Plan(spec, prec, "ecut=5;rows=8").apply_exchange(psi)
    _close(k1, k0, prec)
    _close(e1, e0, prec, True)
    one = hfx.Plan(spec, prec, "ecut=5;tiles=1")
    two = hfx.Plan(spec, prec, "ecut=5;tiles=1;streams=2")
    assert torch.equal(one.apply_exchange(psi)[0], two.apply_exchange(psi)[0])
    parts = [hfx.Plan(spec, prec, "ecut=5;shard=%d/2" % g).apply_exchange(psi) for g in (0, 1)]
    _close(parts[0][0].double() + parts[1][0].double(), k0, prec)
    _close(parts[0][1] + parts[1][1], e0, prec, True)


@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["f32", "f64"])
def test_screened_and_several_systems(prec):
    n, n_orb = 72, 21
    box, psi = _case(n, n, n_orb)
    spec = _spec(n, n, box, n_orb)
    full, red = hfx.Plan(spec, prec), hfx.Plan(spec, prec, "ecut=5")
    a = psi.abs().view(n_orb, -1)
    up = torch.sort((spec.dv * a @ a.T).cpu()[np.triu_indices(n_orb)]).values
    i = up.numel() // 2
    cut = float(0.5 * (up[i] + up[i + 1]))
    assert full.screen(psi, cut) == red.screen(psi, cut)
    (k0, e0), (k1, e1) = full.apply_exchange(psi), red.apply_exchange(psi)
    _close(k1, k0, prec)
    _close(e1, e0, prec, True)

    # two channels of one plan (one size class), and two grids (two classes)
    b = psi[:13].contiguous()
    both = torch.cat([psi.reshape(-1), b.reshape(-1)])
    pair = hfx.Plan([spec, _spec(n, n, box, 13)], prec, "ecut=5;group=1")
    k2, e2 = pair.apply_exchange(both)
    fresh = hfx.Plan(spec, prec, "ecut=5").apply_exchange(psi)
    assert torch.equal(k2[:psi.numel()].view_as(psi), fresh[0])
    other = hfx.Plan(_spec(n, n, box, 13), prec, "ecut=5").apply_exchange(b)
    assert torch.equal(k2[psi.numel():].view_as(b), other[0])
    assert torch.equal(e2, torch.cat([fresh[1], other[1]]))


@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["f32", "f64"])
def test_unequal_box(prec):
    """Bands that differ by axis, and a box whose y band does not fit: the full grid."""
    n = 64
    for box, reduced in (((15.0, 12.0, 14.0), True), ((15.0, 17.5, 14.0), False)):
        psi = torch.from_numpy(generate.random_pw((n, n, n), box, 5, 5.0, 9)).cuda()
        spec = hfx.SystemSpec(n, box, 5)
        red = hfx.Plan(spec, prec, "ecut=5")
        assert ("pair_grid=" in red.describe()) == reduced
        k0, e0 = hfx.Plan(spec, prec).apply_exchange(psi)
        k1, e1 = red.apply_exchange(psi)
        _close(k1, k0, prec)
        _close(e1, e0, prec, True)


def test_named_variant_keeps_the_full_grid():
    box, psi = _case(96, 96, 2)
    spec = _spec(96, 96, box, 2)
    assert "pair_grid=48->72" in hfx.Plan(spec, hfx.FP32, "ecut=5;variant=f32-n96").describe()
    assert "pair_grid" not in hfx.Plan(spec, hfx.FP32, "ecut=5;variant=f32-n96-r").describe()
    assert "pair_grid" not in hfx.Plan(spec, hfx.FP32, "ecut=20").describe()
