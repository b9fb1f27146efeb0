"""Circuits that run as matrix-core blocks are no less accurate than the vector
passes: rms error over three circuits against the same in extended precision.
Layered circuits put the most gates in a block (measured 0.4 of the vector
passes' error in complex64, 0.7 in complex128); the bound is theirs.
"""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu


def _apply(psi, n, g):
    """A U3 or a CNOT in extended precision."""
    v = psi.reshape((2,) * n)
    at = [[slice(None)] * n for _ in range(2)]
    t = g[1] if g[0] == "u" else g[2]
    for b in range(2):
        if g[0] == "cx":
            at[b][n - 1 - g[1]] = 1
        at[b][n - 1 - t] = b
    i0, i1 = tuple(at[0]), tuple(at[1])
    a, b = v[i0].copy(), v[i1].copy()
    u = np.asarray([[0, 1], [1, 0]] if g[0] == "cx" else g[2], dtype=np.complex128).astype(np.clongdouble)
    v[i0], v[i1] = u[0, 0] * a + u[0, 1] * b, u[1, 0] * a + u[1, 1] * b


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n,layers", [(8, 6), (11, 2), (12, 8)])
def test_blocks_err_no_more_than_vector_passes(dt, n, layers):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sq = np.zeros(2)
    for seed in range(3):
        rng = np.random.default_rng(100 * n + seed)
        gates = inputs.probe_layers(rng, n, layers)
        psi = inputs.random_state(rng, n)
        if dt == "c64":
            psi = psi.astype(np.complex64).astype(np.complex128)
        ref = psi.astype(np.clongdouble)
        for g in gates:
            _apply(ref, n, g)
        s = B.State(n, dt)
        for i, kmax in enumerate((0, 13 if dt == "c64" else 12)):
            s.set(psi)
            B.sv_trace_enable(True)
            B.sv_apply_circuit(s.h, gates, kmax)
            assert ("block_build" in B.sv_trace_report()) == (kmax == 0)
            B.sv_trace_enable(False)
            sq[i] += float((np.abs(s.get().astype(np.clongdouble) - ref) ** 2).sum())
        s.close()
    assert sq[0] <= sq[1]
