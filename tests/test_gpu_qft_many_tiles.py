"""Passes of so many small tiles that one launch cannot hold them: a register of
10 qubits on 31 qubits with tiles of at most 8 qubits, and the gradient of 2
qubits on 29.  Reference: the same in double precision, a part of the state at
a time; tolerance: 8 roundings of complex64, relative to a part, which holds at
most 2^-5 of the unit vector's squared norm.
"""
import pytest

from paper_2307_00391_amd import binding as B

pytestmark = pytest.mark.gpu

TOL = 8 * 2.0 ** -24


def _state(torch, n):
    s = B.State(n, "c64")
    torch.manual_seed(n)
    v = torch.view_as_real(s.tensor)
    v.normal_()
    v.mul_((0.5 / (1 << n)) ** 0.5)
    return s


def test_qft_small_tiles_large_state():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, m = 31, 10
    s = _state(torch, n)
    rows = 1 << 16
    v = s.tensor.view(-1, 1 << m)
    at = [0, rows, (v.shape[0] // rows - 1) * rows, (v.shape[0] // rows // 2) * rows]
    ref = [torch.fft.ifft(v[a:a + rows].to(torch.complex128), dim=1, norm="ortho") for a in at]
    B.sv_qft(s.h, 0, m, False, True, 8)
    for a, r in zip(at, ref):
        assert (v[a:a + rows] - r).norm().item() <= TOL * 2.0 ** -2.5
    s.close()


def test_gradient_of_two_qubits_large_state():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, N = 29, 4
    s = _state(torch, n)
    rows = 1 << 20
    v = s.tensor.view(2, -1, N)
    at = [0, rows, v.shape[1] - rows, v.shape[1] // 2]
    k = torch.tensor([0.0, 1.0, 0.0, -1.0], dtype=torch.float64, device="cuda")
    sn, cs = k.abs() / (N // 2 - 1), torch.sqrt(1 - (k / (N // 2 - 1)) ** 2)
    ph = torch.where(k > 0, 1j, torch.where(k < 0, -1j, 1.0 + 0j)).to(torch.complex128)
    ref = []
    for a in at:
        w = torch.fft.fft(v[:, a:a + rows].to(torch.complex128), dim=2, norm="ortho")
        w = torch.stack([ph * (cs * w[0] - sn * w[1]), ph * (sn * w[0] + cs * w[1])])
        ref.append(torch.fft.ifft(w, dim=2, norm="ortho"))
    B.sv_spectral_derivative(s.h, 0, 2, n - 1)
    for a, r in zip(at, ref):
        assert (v[:, a:a + rows] - r).norm().item() <= TOL * 2.0 ** -2.5
    s.close()
