"""SCDM pivots with the lazily downdated blocks of points, where the blocks'
bounds matter most: delocalised orbitals (norms close to each other, so many
blocks stay in play), localised ones (most blocks never come up), and a single
one.  The oracle projects every column in every step."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,L,n_orb", [("pw", 24, 10.0, 1), ("pw", 24, 10.0, 2),
                                            ("pw", 24, 10.0, 65), ("pw", 64, 15.7, 70),
                                            ("g", 64, 15.7, 48), ("white", 24, 10.0, 33)])
def test_pivots_and_orbitals(kind, n, L, n_orb):
    shape, box = (n, n, n), (L, L, L)
    dv = L ** 3 / n ** 3
    if kind == "pw":
        psi = generate.random_pw(shape, box, n_orb, 5.0, 21)
    elif kind == "g":
        psi = generate.gaussians(shape, box, n_orb, 20.0, 22)[0]
    else:
        psi = generate.white_noise(shape, box, n_orb, 23)
    psi, _ = oracle.lowdin(psi, dv)
    piv_ref, gaps = oracle.scdm_pivots(psi)
    assert gaps.min() > 1e-9, gaps.min()
    phi_ref, _ = oracle.scdm(psi, dv)
    plan = hfx.Plan(hfx.SystemSpec(n, box, n_orb), hfx.FP64)
    phi, piv = plan.scdm(torch.from_numpy(psi).cuda())
    assert np.array_equal(piv.cpu().numpy(), piv_ref)
    # float64, n_orb products of unit-norm factors per value: the bar of the
    # parity tests, 1e-10 of the largest value
    assert np.max(np.abs(phi.cpu().numpy() - phi_ref)) <= 1e-10 * np.max(np.abs(phi_ref))
