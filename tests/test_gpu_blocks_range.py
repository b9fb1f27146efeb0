"""Matrix-core blocks over the type's range: states scaled by powers of two down
to denormal amplitudes and up to the largest are no further from extended
precision than by the vector passes, and circuits with a gate that is not
unitary take the vector passes.
"""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu

N = 10


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def _run(dt, psi, gates, kmax):
    s = B.State(N, dt)
    s.set(psi)
    B.sv_trace_enable(True)
    B.sv_apply_circuit(s.h, gates, kmax)
    blocks = "block_build" in B.sv_trace_report()
    B.sv_trace_enable(False)
    out = s.get()
    s.close()
    return out, blocks


def _reference(psi, gates):
    v = psi.astype(np.clongdouble).reshape((2,) * N)
    for g in gates:
        t = g[1] if g[0] == "u" else g[2]
        at = [[slice(None)] * N for _ in range(2)]
        for b in range(2):
            if g[0] == "cx":
                at[b][N - 1 - g[1]] = 1
            at[b][N - 1 - t] = b
        i0, i1 = tuple(at[0]), tuple(at[1])
        a, b = v[i0].copy(), v[i1].copy()
        u = np.asarray([[0, 1], [1, 0]] if g[0] == "cx" else g[2], dtype=np.complex128).astype(np.clongdouble)
        v[i0], v[i1] = u[0, 0] * a + u[0, 1] * b, u[1, 0] * a + u[1, 1] * b
    return v.reshape(-1)


@pytest.mark.parametrize("dt,e", [("c64", e) for e in (-140, -125, -115, -105, 90, 100, 124)] +
                         [("c128", e) for e in (-1060, -1000, 1000, 1010, 1021)])
def test_scaled_states(dt, e):
    gates = inputs.probe_layers(np.random.default_rng(1), N, 2)
    psi = inputs.random_state(np.random.default_rng(2), N)
    if dt == "c64":
        psi = psi.astype(np.complex64).astype(np.complex128)
    psi = psi * 2.0 ** e
    psi = psi.astype(np.complex64).astype(np.complex128) if dt == "c64" else psi
    ref = _reference(psi, gates)
    err = []
    for kmax in (0, 9):
        out, blocks = _run(dt, psi, gates, kmax)
        assert blocks == (kmax == 0)
        err.append(np.linalg.norm(((out.astype(np.clongdouble) - ref) * np.longdouble(2) ** -e).astype(np.complex128)))
    assert err[0] <= err[1]


@pytest.mark.parametrize("dt", ["c128", "c64"])
def test_largest_amplitude(dt):
    R, eps = (np.float64, 2.0 ** -53) if dt == "c128" else (np.float32, 2.0 ** -24)
    gates = inputs.probe_layers(np.random.default_rng(3), N, 2)
    big = float(np.finfo(R).max)
    psi = np.zeros(1 << N, dtype=np.complex128)
    psi[77] = big
    ref = _reference(psi / big, gates)
    out, blocks = _run(dt, psi, gates, 0)
    assert blocks and np.isfinite(out).all()
    assert np.abs(out / big - ref.astype(np.complex128)).max() <= 8 * len(gates) * eps


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("u", [[[1, 0], [0, 0]], [[0.5, 0], [0, 0.5]], [[1, 1], [1, -1]], [[1e30, 0], [0, 1e-30]]])
def test_gates_that_are_not_unitary_take_the_vector_passes(dt, u):
    gates = inputs.probe_layers(np.random.default_rng(4), N, 1) + [("u", 4, u)]
    psi = inputs.random_state(np.random.default_rng(5), N)
    a, blocks = _run(dt, psi, gates, 0)
    b, _ = _run(dt, psi, gates, N)
    assert not blocks
    assert np.array_equal(a, b)
