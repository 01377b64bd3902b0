"""Contractions at the edges of their output tiles (16, 32, 64, 128 orbitals and
the first set of several tiles): the exchange matrix in both precisions, the
symmetric overlap (through Cholesky orthonormalisation) and the |psi||psi|
overlaps of the screening, against numpy float64.

Tolerances: float64 products of nr terms, each factor of unit norm: nr eps in
the worst case, sqrt(nr) eps expected; 64 sqrt(nr) eps is used.  The float32
split product folds 32-term float32 sums: 32 2^-24 of sum |a b| per fold at
worst, so 32 2^-24 of the product of norms bounds the total."""
import numpy as np
import pytest
import torch

from paper_2309_00651_amd import hfx

pytestmark = pytest.mark.gpu

SIZES = (1, 15, 16, 17, 32, 33, 64, 65, 128, 129, 200)


def _orbitals(n_orb, nr, seed):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((n_orb, nr))


@pytest.mark.parametrize("n_orb", SIZES)
@pytest.mark.parametrize("prec", [hfx.FP32, hfx.FP64], ids=["f32", "f64"])
def test_matrix_overlap_and_screen_products(n_orb, prec):
    spec = hfx.SystemSpec((24, 24, 48) if n_orb % 2 else 24, (10.0, 10.0, 10.0), n_orb)
    nr, dv = spec.nr, spec.dv
    eps = np.finfo(float).eps
    psi = _orbitals(n_orb, nr, 5 + n_orb) / np.sqrt(nr * dv)
    w = _orbitals(n_orb, nr, 905 + n_orb) / np.sqrt(nr * dv)
    plan = hfx.Plan(spec, prec)
    p = torch.from_numpy(psi).cuda().view(n_orb, -1)
    k = torch.from_numpy(w).cuda().to(plan.kpsi_dtype)
    wk = k.double().cpu().numpy()
    m = plan.exchange_matrix(p, k).view(n_orb, n_orb).cpu().numpy()
    norms = dv * np.linalg.norm(psi, axis=1)[:, None] * np.linalg.norm(wk, axis=1)[None, :]
    bar = 64 * np.sqrt(nr) * eps if prec == hfx.FP64 else 32 * 2.0 ** -24
    assert np.all(np.abs(m - dv * psi @ wk.T) <= bar * norms)

    # |psi| |psi|^T: every pair decided as numpy decides it, at a cut in the
    # widest gap of the middle half of the overlaps
    a = dv * np.abs(psi) @ np.abs(psi).T
    up = np.sort(a[np.triu_indices(n_orb)])
    if up.size > 8:
        mid = up[up.size // 4: 3 * up.size // 4 + 1]
        g = int(np.argmax(np.diff(mid)))
        cut = 0.5 * (mid[g] + mid[g + 1])
        assert mid[g + 1] - mid[g] > 1e3 * np.sqrt(nr) * eps
        assert plan.screen(p, cut) == [int(np.sum(up >= cut))]
        plan.screen(p, 0.0)

    # S = L L^T of the symmetric product: psi becomes orthonormal
    plan.orthonormalize(p, hfx.ORTHO_CHOLESKY)
    q = p.cpu().numpy().reshape(n_orb, nr)
    s = dv * q @ q.T
    cond = np.linalg.cond(dv * psi @ psi.T)
    assert np.max(np.abs(s - np.eye(n_orb))) <= 64 * np.sqrt(nr) * eps * cond
