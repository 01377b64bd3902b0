"""Reduced pair grids at the orbital counts where their default batches no longer
fit the workspace of the caller's grid: the batches shrink, the workspace stays
within that bound, and the results are the caller's grid's."""
import pytest
import torch

from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu

H = 23.5 / 96


def _spec(n, n_orb):
    return hfx.SystemSpec(n, (n * H,) * 3, n_orb)


@pytest.mark.parametrize("n,prec,counts", [
    (120, hfx.FP64, (112, 113, 256)), (128, hfx.FP64, (112, 113, 256)),
    (108, hfx.FP64, (208, 209)), (120, hfx.FP32, (582, 583)), (64, hfx.FP64, (64, 512))])
def test_pair_grid_within_the_workspace(n, prec, counts):
    for n_orb in counts:
        full = hfx.Plan(_spec(n, n_orb), prec)
        red = hfx.Plan(_spec(n, n_orb), prec, "ecut=5")
        assert "->" in red.describe() and "pair_grid=" not in full.describe()
        assert red.ws_bytes <= full.ws_bytes


def test_results_with_smaller_batches():
    """The bars of the reduced grid's parity test (float64)."""
    n, n_orb = 120, 113
    psi = torch.from_numpy(generate.random_pw((n,) * 3, (n * H,) * 3, 8, 5.0, 7)).cuda()
    # combinations of a few orbitals: inside the same sphere
    gen = torch.Generator(device="cuda").manual_seed(1)
    mix = torch.randn(n_orb, 8, generator=gen, device="cuda", dtype=torch.float64)
    psi = (mix @ psi.view(8, -1)).view(n_orb, n, n, n)
    k0, e0 = hfx.Plan(_spec(n, n_orb), hfx.FP64).apply_exchange(psi)
    red = hfx.Plan(_spec(n, n_orb), hfx.FP64, "ecut=5")
    k1, e1 = red.apply_exchange(psi)
    assert float((k1 - k0).abs().max()) <= 1e-10 * float(k0.abs().max())
    assert float((e1 - e0).abs().max()) <= 1e-12 * float(e0.abs().max())
    # screening and its end rebuild the schedule within the same batches
    before = red.schedule_info()
    red.screen(psi, 1e-300)
    k2 = red.apply_exchange(psi)[0]
    assert float((k2 - k0).abs().max()) <= 1e-10 * float(k0.abs().max())
    red.screen(psi, 0.0)
    assert red.schedule_info() == before
    assert torch.equal(red.apply_exchange(psi)[0], k1)
