"""Mixed circuits whose gates all fit a block of four qubits (at most two
controls on a swap, three on the others), so that they do run as matrix-core
blocks: controlled gates, Toffolis and controlled swaps with controls inside and
outside the tile, on states of one unit per tile up to tiles of half the state;
and the same circuits with a gate of five qubits, which take the vector passes.
Tolerance: 8 roundings per gate in relative l2, as both executors round each
amplitude a few times per gate.
"""
import numpy as np
import pytest

import oracle
from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu

EPS = {"c128": 2.0 ** -53, "c64": 2.0 ** -24}
X = np.array([[0, 1], [1, 0]], dtype=np.complex128)


def _apply(psi, g):
    if g[0] == "u":
        oracle.apply_gate(psi, g[1], g[2], *g[3:5])
    elif g[0] == "x":
        oracle.apply_gate(psi, g[1], X, *g[2:4])
    else:
        oracle.apply_swap(psi, g[1], g[2], *g[3:5])


def _mixed(rng, n, count):
    out = []
    for g in inputs.random_circuit(rng, n, count, max_ctrls=2):
        out.append(g)
        if len(out) % 6 == 0:
            q = [int(v) for v in rng.permutation(n)[:4]]
            vals = [int(v) for v in rng.integers(0, 2, 3)]
            out.append(("u", q[0], inputs.random_unitary(rng, 2), q[1:], vals) if len(out) % 4 else ("x", q[0], q[1:], vals))
    return out


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n", [8, 9, 11, 14, 16, 18])
@pytest.mark.parametrize("wide", [False, True])
def test_mixed_circuits_as_blocks(dt, n, wide):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(31 * n + wide)
    gates = _mixed(rng, n, 96)
    if wide:
        q = [int(v) for v in rng.permutation(n)[:5]]
        gates.insert(50, ("u", q[0], inputs.random_unitary(rng, 2), q[1:], [1, 0, 1, 1]))
    psi = inputs.random_state(rng, n)
    if dt == "c64":
        psi = psi.astype(np.complex64).astype(np.complex128)
    s = B.State(n, dt)
    s.set(psi)
    B.sv_trace_enable(True)
    B.sv_apply_circuit(s.h, gates)
    assert ("block_build" in B.sv_trace_report()) == (not wide)
    B.sv_trace_enable(False)
    got = s.get()
    s.close()
    for g in gates:
        _apply(psi, g)
    assert np.linalg.norm(got - psi) <= 8 * len(gates) * EPS[dt]
