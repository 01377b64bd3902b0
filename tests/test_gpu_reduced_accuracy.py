"""Reduced pair grids lose nothing against the caller's grid.

float64: K psi of both against 80-bit arithmetic.  The orbitals are synthesised in 80 bits and
rounded once, so what they hold outside the declared band is one rounding.  Both
paths round the same transforms; the reduced one rounds psi and K psi three
times more each (six times 2^-53 / sqrt(3), 1.6e-16 together, on the caller's
grid's 2.5e-16), hence the bar of 1.5 times its error.

float32: E_x of both against float64, where the error is the transforms' bias:
no larger on the reduced grid, or below 1e-9 (two codelets in each of six passes,
each biased by at most 2.5e-10 in amplitude, of either sign); and K psi, no
further off than on the caller's grid."""
import numpy as np
import pytest
import torch

from paper_2309_00651_amd import hfx

pytestmark = pytest.mark.gpu

LD = np.longdouble
H = 23.5 / 96
PI = LD("3.14159265358979323846264338327950288")


def _orbitals(n, n_orb):
    """Random plane waves of 5 Ha, 80 bits."""
    g = 2 * np.pi * np.fft.fftfreq(n, 1 / n) / (n * H)
    g2 = g[:, None, None] ** 2 + g[None, :, None] ** 2 + g[None, None, : n // 2 + 1] ** 2
    rng = np.random.default_rng(n)
    c = rng.standard_normal((n_orb, *g2.shape)) + 1j * rng.standard_normal((n_orb, *g2.shape))
    c *= np.exp(-g2 / 8) * (0.5 * g2 <= 5.0)
    psi = np.fft.irfftn(c.astype(np.clongdouble), s=(n, n, n), axes=(1, 2, 3))
    return psi / np.sqrt((psi ** 2).sum((1, 2, 3), keepdims=True) * H ** 3)


def _reduced(n, prec):
    """Plan options that ask for the reduced grid at any orbital count."""
    return "ecut=5;variant=" + hfx.variants(n, prec)[0]


def _kpsi(psi, n):
    g = 2 * PI * np.round(np.fft.fftfreq(n, 1 / n)).astype(LD) / (n * LD(H))
    g2 = g[:, None, None] ** 2 + g[None, :, None] ** 2 + g[None, None, : n // 2 + 1] ** 2
    rc = np.cbrt(3 * (n * LD(H)) ** 3 / (4 * PI))
    safe = np.where(g2 > 0, g2, 1)
    v = np.where(g2 > 0, 8 * PI * np.sin(rc * np.sqrt(safe) / 2) ** 2 / safe, 2 * PI * rc * rc)
    out = np.zeros_like(psi)
    for i in range(len(psi)):
        for j in range(i, len(psi)):
            w = np.fft.irfftn(np.fft.rfftn(psi[i] * psi[j], axes=(0, 1, 2)) * v, s=(n, n, n), axes=(0, 1, 2))
            out[i] -= w * psi[j]
            if j != i:
                out[j] -= w * psi[i]
    return out


@pytest.mark.parametrize("n", [64, 80])
def test_float64_kpsi_is_as_accurate_as_on_the_callers_grid(n):
    psi = _orbitals(n, 6).astype(np.float64)
    ref = _kpsi(psi.astype(LD), n)
    x = torch.from_numpy(psi).cuda()
    err = []
    for options in (None, _reduced(n, hfx.FP64)):
        plan = hfx.Plan(hfx.SystemSpec(n, (n * H,) * 3, 6), hfx.FP64, options)
        assert ("->" in plan.describe()) == (options is not None)
        d = plan.apply_exchange(x)[0].cpu().numpy().astype(LD) - ref
        err.append(float(np.sqrt((d ** 2).sum() / (ref ** 2).sum())))
    assert err[1] <= 1.5 * err[0], err


@pytest.mark.parametrize("n", [64, 108])
def test_scales_of_the_split_products(n):
    """A power of two passes through the split products unchanged; an empty and a
    very small orbital do no harm to the ordinary ones beside them."""
    n_orb = 9
    x = torch.from_numpy(_orbitals(n, n_orb).astype(np.float64)).cuda()
    plan = hfx.Plan(hfx.SystemSpec(n, (n * H,) * 3, n_orb), hfx.FP64, _reduced(n, hfx.FP64))
    assert "->" in plan.describe()
    k = plan.apply_exchange(x)[0]
    for e in (60, -60):
        assert torch.equal(plan.apply_exchange(x * 2.0 ** e)[0], k * 2.0 ** (3 * e))
    y = x.clone()
    y[3] = 0.0
    y[5] *= 1e-290
    z = plan.apply_exchange(y)[0]
    assert torch.isfinite(z).all()
    rest = [a for a in range(n_orb) if a not in (3, 5)]
    few = hfx.Plan(hfx.SystemSpec(n, (n * H,) * 3, len(rest)), hfx.FP64)
    want = few.apply_exchange(x[rest].contiguous())[0]
    assert float((z[rest] - want).abs().max()) <= 1e-14 * float(want.abs().max())


@pytest.mark.parametrize("kernel,w", [(hfx.TRUNCATED, 0.0), (hfx.ERFC, 0.106)], ids=["truncated", "erfc"])
@pytest.mark.parametrize("n", [64, 72, 80, 96, 108, 120, 128])
def test_float32_energy_is_as_accurate_as_on_the_callers_grid(n, kernel, w):
    x = torch.from_numpy(_orbitals(n, 9).astype(np.float64)).cuda()
    spec = hfx.SystemSpec(n, (n * H,) * 3, 9, kernel, w)
    ref = hfx.Plan(spec, hfx.FP64).exchange_energy(x)
    err = [abs(float(((hfx.Plan(spec, hfx.FP32, o).exchange_energy(x) - ref) / ref)[0]))
           for o in (None, _reduced(n, hfx.FP32))]
    assert err[1] <= max(err[0], 1e-9), err


@pytest.mark.parametrize("rho_cut", [0.0, 0.3])
@pytest.mark.parametrize("n", [64, 108])
def test_float32_kpsi_is_as_accurate_as_on_the_callers_grid(n, rho_cut):
    """Screened too (some own pairs, int psi_a^2 = 1, are then the only ones of their row)."""
    n_orb = 21
    x = torch.from_numpy(_orbitals(n, n_orb).astype(np.float64)).cuda()
    x[4] *= 0.5  # its own pair, 0.25, is screened out
    spec = hfx.SystemSpec(n, (n * H,) * 3, n_orb)
    out, kept = [], []
    for prec, options in ((hfx.FP64, None), (hfx.FP32, None), (hfx.FP32, _reduced(n, hfx.FP32))):
        plan = hfx.Plan(spec, prec, options)
        if rho_cut:
            kept.append(plan.screen(x, rho_cut))
        out.append(plan.apply_exchange(x)[0].double())
    assert len({k[0] for k in kept}) <= 1
    err = [float((o - out[0]).norm() / out[0].norm()) for o in out[1:]]
    assert err[1] <= err[0], err
