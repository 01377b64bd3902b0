"""SCDM on non-finite orbitals (a diverged step): no pivot leaves the grid, the
localised orbitals come out non-finite, and a point that holds a NaN is passed
over without hiding the points beside it."""
import pytest
import torch

from paper_2309_00651_amd import hfx

pytestmark = pytest.mark.gpu

N, H = 24, 10.0 / 24


def _orbitals(n_orb):
    gen = torch.Generator(device="cuda").manual_seed(5)
    psi = torch.randn(n_orb, N, N, N, generator=gen, device="cuda", dtype=torch.float64)
    plan = hfx.Plan(hfx.SystemSpec(N, (10.0,) * 3, n_orb), hfx.FP64)
    return plan, plan.orthonormalize(psi)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")], ids=["nan", "inf"])
@pytest.mark.parametrize("n_orb", [1, 8, 70])
def test_a_non_finite_orbital(n_orb, bad):
    plan, psi = _orbitals(n_orb)
    psi[n_orb // 2] = bad
    phi, piv = plan.scdm(psi)
    assert not torch.isfinite(phi).any()
    assert int(piv.min()) >= 0 and int(piv.max()) < N ** 3


@pytest.mark.parametrize("n_orb", [8, 70])
def test_points_beside_a_nan_are_still_candidates(n_orb):
    """The NaN sits at a point of the first pivot's block of 256; the pivots are
    those of the orbitals with zeros at that point."""
    plan, psi = _orbitals(n_orb)
    flat = psi.view(n_orb, -1)
    first = int(flat.square().sum(0).argmax())
    at = first // 256 * 256 + (0 if first % 256 else 1)
    clean = psi.clone()
    clean.view(n_orb, -1)[:, at] = 0.0
    flat[0, at] = float("nan")
    want = plan.scdm(clean)[1]
    assert int(want[0]) == first
    phi, piv = plan.scdm(psi)
    assert torch.equal(piv, want)
    assert not torch.isfinite(phi).any()
