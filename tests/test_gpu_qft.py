"""GPU parity of the multi-pass QFT and the fused spectral gradient at the
edges of their tiles: registers that fill one tile exactly, one qubit more,
two and three groups, mirrored middle bits of width 0, 1 and more, registers
off the bottom of the state, and states smaller than a tile.

Reference: numpy's FFT in double precision.  Tolerance: an FFT's relative l2
error grows no faster than a small multiple of the unit roundoff per stage; 4
per stage covers the butterflies, the twiddle's own rounding and its product.
"""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B

pytestmark = pytest.mark.gpu

EPS = {"c128": 2.0 ** -53, "c64": 2.0 ** -24}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def _psi(n, dt, seed):
    rng = np.random.default_rng(seed)
    v = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    v /= np.linalg.norm(v)
    return v.astype(np.complex64).astype(np.complex128) if dt == "c64" else v


def _bitrev(m):
    r = np.zeros(1 << m, dtype=np.int64)
    for j in range(m):
        r |= ((np.arange(1 << m) >> j) & 1) << (m - 1 - j)
    return r


def _ref(psi, lo, m, inverse, swaps):
    v = psi.reshape(-1, 1 << m, 1 << lo)
    if inverse:
        v = v if swaps else v[:, _bitrev(m)]
        return np.fft.fft(v, axis=1, norm="ortho").reshape(-1)
    v = np.fft.ifft(v, axis=1, norm="ortho")
    return (v if swaps else v[:, _bitrev(m)]).reshape(-1)


def _close(got, ref, dt, m):
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert err <= 4 * (m + 2) * EPS[dt], err


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n,lo,m,kmax", [
    (1, 0, 1, 0), (2, 0, 2, 0), (3, 1, 2, 0), (4, 0, 3, 0), (5, 4, 1, 0),          # below or at one line
    (13, 0, 13, 0), (14, 0, 14, 0), (15, 1, 14, 0), (16, 0, 16, 0), (17, 4, 12, 0),  # one tile, one more
    (9, 0, 9, 6), (12, 2, 9, 6), (13, 3, 10, 7), (11, 0, 11, 7),                    # many groups, middle bits 0, 1, 3
    (21, 0, 21, 0), (20, 3, 17, 0), (19, 6, 12, 0)])
def test_qft_against_fft(dt, n, lo, m, kmax):
    psi = _psi(n, dt, 40 * n + m)
    for inverse in (False, True):
        for swaps in (False, True):
            s = B.State(n, dt)
            s.set(psi)
            B.sv_qft(s.h, lo, m, inverse, swaps, kmax)
            _close(s.get(), _ref(psi, lo, m, inverse, swaps), dt, m)
            s.close()


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n,lo,m,anc,kmax", [
    (3, 0, 2, 2, 0), (4, 1, 3, 0, 0), (6, 4, 2, 1, 0), (14, 0, 12, 13, 0), (14, 1, 13, 0, 0), (15, 0, 13, 14, 0),
    (16, 2, 12, 15, 0), (17, 3, 13, 1, 0), (12, 2, 8, 11, 6), (13, 4, 8, 2, 7), (20, 0, 19, 19, 0)])
def test_spectral_against_fft(dt, n, lo, m, anc, kmax):
    psi = _psi(n, dt, 50 * n + m)
    s = B.State(n, dt)
    s.set(psi)
    B.sv_spectral_derivative(s.h, lo, m, anc, kmax)
    got = s.get()
    s.close()
    N = 1 << m
    v = np.fft.fft(psi.reshape(-1, N, 1 << lo), axis=1, norm="ortho").reshape(-1)
    idx = np.arange(1 << n)
    i0 = idx[(idx >> anc & 1) == 0]
    i1 = i0 | (1 << anc)
    k = (i0 >> lo) & (N - 1)
    kp = np.where(k < N // 2, k, k - N).astype(float)
    kp[k == N // 2] = 0
    sn = np.abs(kp) / (N // 2 - 1)
    cs = np.sqrt(1 - sn * sn)
    ph = np.where(kp > 0, 1j, np.where(kp < 0, -1j, 1))
    a0, a1 = v[i0], v[i1]
    v[i0], v[i1] = ph * (cs * a0 - sn * a1), ph * (sn * a0 + cs * a1)
    ref = np.fft.ifft(v.reshape(-1, N, 1 << lo), axis=1, norm="ortho").reshape(-1)
    _close(got, ref, dt, 2 * m)
