"""Row products with two, three and four row wavefronts (129 to 512 orbitals), in
place (Loewdin, float64) and from float32 sources (ACE projectors), against the
oracle's Loewdin and a float64 product; the bars of the parity tests of both."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_00651_amd import hfx

pytestmark = pytest.mark.gpu

N = 24


@pytest.mark.parametrize("n_orb", [129, 257, 385, 400, 512])
def test_in_place_and_float32_sources(n_orb):
    rng = np.random.default_rng(n_orb)
    psi = rng.standard_normal((n_orb, N, N, N))
    dv = 1000.0 / N ** 3
    spec = hfx.SystemSpec(N, (10.0,) * 3, n_orb)
    ref, lam = oracle.lowdin(psi, dv)
    assert lam > 1e-3
    got = hfx.Plan(spec, hfx.FP64).orthonormalize(torch.from_numpy(psi).cuda())
    assert np.max(np.abs(got.cpu().numpy() - ref)) <= 1e-11 * np.max(np.abs(ref))
    # any W and positive definite -M give projectors: rows of L^(-1) W
    w = torch.from_numpy(psi.astype(np.float32)).cuda()
    m = -torch.from_numpy(dv * (ref.reshape(n_orb, -1) @ ref.reshape(n_orb, -1).T)
                          + np.diag(np.linspace(0.0, 1.0, n_orb))).cuda()
    p = hfx.Plan(spec, hfx.FP32).ace_build(w, m.contiguous())
    low = np.linalg.cholesky(-m.cpu().numpy())
    want = np.linalg.solve(low, w.double().cpu().numpy().reshape(n_orb, -1))
    assert np.max(np.abs(p.cpu().numpy().reshape(n_orb, -1) - want)) <= 1e-11 * np.max(np.abs(want))
