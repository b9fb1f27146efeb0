"""A transform keeps amplitudes of up to 2^-1.5 of the type's largest number
finite where its result is: four equal amplitudes of one radix step, and the
transform back.  The error is at most 16 roundings of the largest amplitude.
"""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n,lo,m", [(10, 0, 10), (12, 3, 4), (16, 0, 16), (16, 5, 11)])
@pytest.mark.parametrize("swaps", [True, False])
def test_large_amplitudes_stay_finite(dt, n, lo, m, swaps):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    R, eps = (np.float64, 2.0 ** -53) if dt == "c128" else (np.float32, 2.0 ** -24)
    big = float(np.finfo(R).max) * 2.0 ** -1.5
    psi = np.zeros(1 << n, dtype=np.complex128)
    q = 1 << (lo + m - 2)                       # the top two register bits
    psi[[0, q, 2 * q, 3 * q]] = big
    s = B.State(n, dt)
    s.set(psi)
    B.sv_qft(s.h, lo, m, False, swaps)
    assert np.isfinite(s.get()).all()
    B.sv_qft(s.h, lo, m, True, swaps)
    assert np.abs(s.get() / big - psi / big).max() <= 16 * eps
    s.close()
