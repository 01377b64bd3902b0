"""Rows per tile pair of screened plans: 32 where that makes the tile pairs enough
fewer for the grid, 16 otherwise, by the tile pairs of both (named) choices; the
results are those of the choice by name (its batches may hold more tile pairs, so
float32 sums run in another order: n 2^-24 of the largest K psi)."""
import pytest
import torch

from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu

NEED = {64: 1.52, 72: 1.52, 80: 1.3, 96: 1.15, 108: 0.0}


@pytest.mark.parametrize("share", [0.03, 0.25, 1.0])
@pytest.mark.parametrize("n,n_orb", [(64, 85), (72, 41), (80, 64), (96, 40), (108, 33)])
def test_rows_follow_the_tile_pairs(n, n_orb, share):
    box = (n * 23.5 / 96,) * 3
    psi = torch.from_numpy(generate.gaussians((n,) * 3, box, n_orb, 20.0, 5)[0]).cuda()
    spec = hfx.SystemSpec(n, box, n_orb, hfx.ERFC, 0.106)
    a = psi.abs().view(n_orb, -1)
    i, j = torch.triu_indices(n_orb, n_orb)
    overlaps = (spec.dv * (a @ a.T)).cpu()[i, j].sort().values
    at = int((1 - share) * (len(overlaps) - 1))
    cut = float(0.5 * (overlaps[at] + overlaps[at + 1])) if share < 1 else 1e-300
    plans = [hfx.Plan(spec, hfx.FP32, "ecut=20" + o) for o in ("", ";rows=16", ";rows=32")]
    kept = {p.screen(psi, cut)[0] for p in plans}
    assert len(kept) == 1
    low, tall = (p.schedule_info()[1] for p in plans[1:])
    rows = 32 if low >= NEED[n] * tall else 16
    assert " rows=%d " % rows in plans[0].describe()
    named = plans[2 if rows == 32 else 1]
    assert plans[0].schedule_info()[1:] == named.schedule_info()[1:]
    (k, e), (k1, e1) = plans[0].apply_exchange(psi), named.apply_exchange(psi)
    assert float((k - k1).abs().max()) <= n_orb * 2.0 ** -24 * float(k1.abs().max())
    assert abs(float((e - e1) / e1)) <= 1e-12
