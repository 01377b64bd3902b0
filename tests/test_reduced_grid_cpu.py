"""The identities behind the reduced pair grids, checked with numpy at every
compiled triple (points n, sampling points n / 2, pair-grid points m) and at
the widest band k that the dispatch rule accepts, 2 k + 1 <= n / 2 and
3 k + 1 <= m: pair densities (band k) from every other point, potentials on m
points, orbitals resampled n -> m and K psi (band 3 k / 2) m -> n with the
closed-form matrices.  One axis at a time: the three axes of the path are
independent products."""
import numpy as np
import pytest

AXES = [(64, 48), (72, 60), (80, 60), (96, 72), (108, 80), (120, 96), (128, 96)]


def _resample(a, b, kmax):
    """R[i][j] = sin((2 kmax + 1) pi d / ab) / (a sin(pi d / ab)), d = i a - j b."""
    d = (np.arange(b)[:, None] * a - np.arange(a)[None, :] * b) % (a * b)
    num, den = np.sin(np.pi * ((2 * kmax + 1) * d % (2 * a * b)) / (a * b)), np.sin(np.pi * d / (a * b))
    return np.where(d == 0, (2 * kmax + 1) / a, num / np.where(d == 0, 1.0, a * den))


def _orbitals(n, band, rng, count=4):
    c = np.zeros((count, n // 2 + 1), complex)
    c[:, : band + 1] = rng.standard_normal((count, band + 1)) + 1j * rng.standard_normal((count, band + 1))
    c[:, 0] = c[:, 0].real
    return np.fft.irfft(c, n, axis=1) * n


def _kpsi_full(psi, v):
    n = psi.shape[1]
    out = np.zeros_like(psi)
    for a in range(len(psi)):
        for b in range(len(psi)):
            out[a] -= psi[b] * np.fft.ifft(v(np.fft.fftfreq(n, 1 / n)) * np.fft.fft(psi[a] * psi[b])).real
    return out


def _kpsi_reduced(psi, v, k, m):
    n = psi.shape[1]
    h = n // 2
    samp, red = psi[:, ::2], psi @ _resample(n, m, k // 2).T
    out = np.zeros_like(red)
    f = np.fft.fftfreq(h, 1 / h).astype(int)
    keep = np.abs(f) <= k
    for a in range(len(psi)):
        for b in range(len(psi)):
            g = np.zeros(m, complex)
            g[f[keep]] = (v(f) * np.fft.fft(samp[a] * samp[b]) / h)[keep]
            out[a] -= red[b] * (np.fft.ifft(g) * m).real
    return out @ _resample(m, n, k + k // 2).T


def _widest(n, m):
    return max(k for k in range(0, n, 2) if 2 * k + 1 <= n // 2 and 3 * k + 1 <= m)


@pytest.mark.parametrize("n,m", AXES)
def test_reduced_grid_gives_the_full_grids_kpsi(n, m):
    v = lambda q: 1.0 / (1.0 + 0.05 * q * q)
    rng = np.random.default_rng(n)
    k = _widest(n, m)
    for band in (k, 0, 2):
        psi = _orbitals(n, band // 2, rng)
        ref = _kpsi_full(psi, v)
        assert np.max(np.abs(_kpsi_reduced(psi, v, band, m) - ref)) <= 1e-12 * np.max(np.abs(ref))
    # one step beyond the rule the products alias: far above the rounding bar
    psi = _orbitals(n, k // 2 + 1, rng)
    ref = _kpsi_full(psi, v)
    assert np.max(np.abs(_kpsi_reduced(psi, v, k + 2, m) - ref)) > 1e-10 * np.max(np.abs(ref))
