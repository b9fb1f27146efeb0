"""Gate circuits as matrix-core blocks (sv_apply_circuit with max_local = 0)
against the oracle and against the vector passes (max_local > 0), at the edges
of the planner and of the tiles: states of one block unit, tiles with fewer
units than wavefronts, controls outside the tile, diagonal gates, gates of four
qubits, and states with infinite or NaN amplitudes.

Tolerance: a block's results are sums of 16 products, each within a rounding of
the type; per gate the vector passes are allowed the same, so 8 roundings per
gate in relative l2 cover both.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu

EPS = {"c128": 2.0 ** -53, "c64": 2.0 ** -24}
X = np.array([[0, 1], [1, 0]], dtype=np.complex128)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def _apply(psi, g):
    if g[0] == "u":
        oracle.apply_gate(psi, g[1], g[2], *(g[3:5] if len(g) > 3 else ((), None)))
    elif g[0] == "x":
        oracle.apply_gate(psi, g[1], X, *(g[2:4] if len(g) > 2 else ((), None)))
    elif g[0] == "cx":
        oracle.apply_gate(psi, g[2], X, [g[1]], [1])
    else:
        oracle.apply_swap(psi, g[1], g[2], *(g[3:5] if len(g) > 3 else ((), None)))


def _phases(rng, n, count):
    """Diagonal gates: with and without controls, both entries different from 1."""
    out = []
    for i in range(count):
        qs = [int(q) for q in rng.permutation(n)[:4]]
        nc = i % 4
        d = np.diag(np.exp(1j * rng.uniform(0, 2 * math.pi, 2)))
        out.append(("u", qs[0], d, qs[1:1 + nc], [int(v) for v in rng.integers(0, 2, nc)]))
    return out


def _circuit(kind, rng, n):
    if kind == "layers":
        return inputs.probe_layers(rng, n, 3)
    if kind == "mixed":
        return inputs.random_circuit(rng, n, 48, max_ctrls=3)
    if kind == "phases":
        return _phases(rng, n, 24) + inputs.random_circuit(rng, n, 8) + _phases(rng, n, 8)
    return [("u", n - 1, inputs.random_unitary(rng, 2), [0, 1, n // 2], [1, 0, 1])]      # one gate, three controls


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("kind", ["layers", "mixed", "phases", "one"])
@pytest.mark.parametrize("n", [7, 8, 9, 11, 14, 16, 19])
def test_blocks_match_oracle_and_vector_passes(dt, kind, n):
    rng = np.random.default_rng(77 * n + len(kind))
    gates = _circuit(kind, rng, n)
    psi = inputs.random_state(rng, n)
    if dt == "c64":
        psi = psi.astype(np.complex64).astype(np.complex128)
    ref = psi.copy()
    for g in gates:
        _apply(ref, g)
    tol = 8 * len(gates) * EPS[dt]
    for kmax in (0, min(n, 9)):
        s = B.State(n, dt)
        s.set(psi)
        B.sv_apply_circuit(s.h, gates, kmax)
        err = np.linalg.norm(s.get() - ref)
        s.close()
        assert err <= tol, (kmax, err)


@pytest.mark.parametrize("dt,k,c", [("c64", 13, 3), ("c64", 13, 4), ("c64", 11, 3), ("c128", 12, 2), ("c128", 12, 3)])
def test_blocks_pinned_tiles(dt, k, c):
    """Every tile the tuner can pick, through the tuning entry it would store."""
    n = 22
    rng = np.random.default_rng(5 * k + c)
    gates = inputs.random_circuit(rng, n, 24) + inputs.probe_layers(rng, n, 1)
    psi = inputs.random_state(rng, n)
    if dt == "c64":
        psi = psi.astype(np.complex64).astype(np.complex128)
    ref = psi.copy()
    for g in gates:
        _apply(ref, g)
    s = B.State(n, dt)
    s.set(psi)
    before = set(ln.split()[0] for ln in B.sv_tune_report().splitlines() if ln.startswith("fused/"))
    B.sv_apply_circuit(s.h, gates, 0)
    key = [ln.split()[0] for ln in B.sv_tune_report().splitlines() if ln.startswith("fused/") and ln.split()[0] not in before]
    keys = key or [ln.split()[0] for ln in B.sv_tune_report().splitlines() if ln.startswith(f"fused/{dt}/{n}/")]
    try:
        for q in keys:
            B.sv_tune_set(q, [k, c, 1])
        s.set(psi)
        B.sv_apply_circuit(s.h, gates, 0)
        assert np.linalg.norm(s.get() - ref) <= 8 * len(gates) * EPS[dt]
    finally:
        for q in keys:
            B.sv_tune_set(q, [])
        s.close()


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_non_finite_amplitudes_spread_no_further(dt, bad):
    """The amplitudes that stay finite are those the vector passes keep finite,
    with the same values."""
    n = 12
    rng = np.random.default_rng(12)
    u = [inputs.random_unitary(rng, 2) for _ in range(4)]
    gates = [("u", 2, u[0]), ("cx", 2, 5), ("u", 7, u[1], [9], [1]), ("x", 3), ("u", 5, u[2], [11, 0], [1, 1]),
             ("swap", 1, 10), ("u", 4, np.diag([1.0, np.exp(0.4j)]))]
    psi = inputs.random_state(rng, n)
    psi[1234] = bad
    got = []
    for kmax in (0, 9):
        s = B.State(n, dt)
        s.set(psi)
        B.sv_apply_circuit(s.h, gates, kmax)
        got.append(s.get())
        s.close()
    fin = [np.isfinite(g.real) & np.isfinite(g.imag) for g in got]
    assert np.array_equal(fin[0], fin[1])
    assert 1 <= (~fin[0]).sum() < 64
    assert np.abs(got[0][fin[0]] - got[1][fin[0]]).max() <= 64 * EPS[dt]
