"""A first call tunes its launch parameters; what that costs stays in proportion
to the call.  The bounds are about three times what is measured (a dense unitary
of 10 qubits on 24: 13 calls' time)."""
import time

import pytest

from paper_2307_00391_amd import binding as B

pytestmark = pytest.mark.gpu


def _first_and_steady(torch, call, forget):
    call()                                   # the kernels are loaded
    forget()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    call()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(3):
        call()
    torch.cuda.synchronize()
    return t1 - t0, (time.perf_counter() - t1) / 3


def test_dense_unitary_of_half_a_millisecond():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, m = 24, 10
    s = B.State(n, "c64")
    B.sv_init_basis(s.h, 1 << (n - 1))
    U = torch.eye(1 << m, dtype=torch.complex64, device="cuda")
    first, steady = _first_and_steady(torch, lambda: B.sv_apply_ctrl_unitary(s.h, U, 0, m, n - 1),
                                      lambda: B.sv_tune_set(f"cgemm/c64/{1 << (n - 1 - m)}/{1 << m}/{1 << m}/0", []))
    s.close()
    assert first <= 40 * steady
