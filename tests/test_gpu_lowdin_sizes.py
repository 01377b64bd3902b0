"""Loewdin orthonormalisation around the sizes where its S^(-1/2) changes hands
(one workgroup up to 64 orbitals, launches above; 16 x 16 blocks inside),
against the float64 eigendecomposition.  Both are float64: the difference is
bounded by eps times a few sums of n terms and the conditioning of S, 1e-11 at
these sizes and condition numbers below 100."""
import numpy as np
import pytest
import torch

from paper_2309_00651_amd import hfx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_orb", [1, 2, 15, 16, 17, 48, 63, 64, 65, 96, 130])
def test_lowdin_matches_eigendecomposition(n_orb):
    spec = hfx.SystemSpec(24, (10.0, 10.0, 10.0), n_orb)
    rng = np.random.default_rng(n_orb)
    psi = rng.standard_normal((n_orb, spec.nr)) / np.sqrt(spec.nr * spec.dv)
    mix = np.eye(n_orb) + 0.5 * rng.standard_normal((n_orb, n_orb)) / np.sqrt(n_orb)
    psi = mix @ psi  # overlapping, as an orbital update leaves them
    s = spec.dv * psi @ psi.T
    w, u = np.linalg.eigh(s)
    assert w[-1] / w[0] < 100
    ref = (u / np.sqrt(w)) @ u.T @ psi
    p = torch.from_numpy(psi).cuda()
    plan = hfx.Plan(spec, hfx.FP32)
    plan.orthonormalize(p)
    got = p.cpu().numpy().copy()
    assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))
    plan.orthonormalize(p)  # orthonormal input stays as it is
    assert np.max(np.abs(p.cpu().numpy() - got)) <= 1e-11 * np.max(np.abs(ref))
