"""float64 exchange_energy, which sums v(G) |rho(G)|^2 instead of forming the
potentials, against the energy that apply_exchange sums over them: every grid
(planes in LDS, split planes, slab cells), ragged tiles with diagonal pairs,
band-limited and screened plans, two batch streams.  Both are float64 sums of
the same energies: 1e-12 relative, the parity tests' bar."""
import pytest
import torch

from paper_2309_00651_amd import hfx
from workloads import generate

pytestmark = pytest.mark.gpu

GRIDS = [(24, 24), (24, 48), (64, 64), (64, 128), (72, 72), (80, 80), (96, 96), (108, 108),
         (120, 120), (128, 128)]


def _psi(n, nz, box, n_orb, ecut=5.0):
    return torch.from_numpy(generate.random_pw((nz, n, n), box, n_orb, ecut, 31)).cuda()


def _check(plan, psi):
    e = plan.apply_exchange(psi)[1]
    assert float(((plan.exchange_energy(psi) - e) / e).abs().max()) <= 1e-12


@pytest.mark.parametrize("n,nz", GRIDS)
def test_energy_alone_equals_apply(n, nz):
    h = 10.0 / 24 if n == 24 else 23.5 / 96
    box = (n * h, n * h * 1.05, nz * h)
    for n_orb in (1, 11) if n <= 80 else (3,):
        psi = _psi(n, nz, box, n_orb)
        spec = hfx.SystemSpec((n, n, nz) if n != nz else n, box, n_orb, hfx.ERFC, 0.106)
        for opts in (None, "ecut=20", "ecut=5"):
            if n == 24 and opts:
                continue
            _check(hfx.Plan(spec, hfx.FP64, opts), psi)


def test_screened_and_streams():
    n, n_orb, box = 64, 37, (15.0, 15.5, 16.0)
    psi = _psi(n, n, box, n_orb)
    spec = hfx.SystemSpec(n, box, n_orb)
    for opts in ("ecut=20;tiles=1;streams=2", "ecut=20"):
        plan = hfx.Plan(spec, hfx.FP64, opts)
        _check(plan, psi)
        plan.screen(psi, 0.6)
        _check(plan, psi)


def test_several_systems_and_graph():
    box = (10.0,) * 3
    specs = [hfx.SystemSpec(24, box, k) for k in (5, 9)]
    psi = torch.cat([_psi(24, 24, box, k).reshape(-1) for k in (5, 9)])
    plan = hfx.Plan(specs, hfx.FP64)
    _check(plan, psi)
    e = plan.exchange_energy(psi)
    out = torch.empty_like(e)
    g = plan.graph(hfx.GRAPH_ENERGY, psi, ex=out)
    for _ in range(3):
        out.zero_()
        g.launch()
        assert torch.equal(out, e)
