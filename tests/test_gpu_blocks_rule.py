"""Which circuits below 22 qubits run as matrix-core blocks: those with enough
dense gates, not those of phases, NOTs and swaps with a dense gate or two."""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu


def _phases(rng, n, count, dense):
    out = []
    for _ in range(count):
        q = [int(v) for v in rng.permutation(n)[:2]]
        out.append(("u", q[0], np.diag([1.0, np.exp(1j * rng.uniform(0, 6))]), q[1:], [1]))
    return out + [("u", int(rng.integers(0, n)), inputs.random_unitary(rng, 2)) for _ in range(dense)]


@pytest.mark.parametrize("dt,n,kind,blocks", [
    ("c64", 14, "layers8", True), ("c128", 14, "layers8", True), ("c64", 18, "mixed80", True), ("c64", 20, "layers4", True),
    ("c128", 21, "phases60+1", False), ("c64", 21, "phases60+1", False), ("c64", 14, "mixed16", False),
    ("c128", 21, "mixed80", False), ("c64", 12, "layers1", False), ("c64", 8, "mixed4", False)])
def test_route(dt, n, kind, blocks):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(10 * n + 1)
    if kind.startswith("layers"):
        gates = inputs.probe_layers(rng, n, int(kind[6:]))
    elif kind.startswith("mixed"):
        gates = inputs.random_circuit(rng, n, int(kind[5:]))
    else:
        a, d = kind[6:].split("+")
        gates = _phases(rng, n, int(a), int(d))
    s = B.State(n, dt)
    out = []
    for kmax in (0, 12):
        B.sv_init_basis(s.h, 3)
        B.sv_trace_enable(True)
        B.sv_apply_circuit(s.h, gates, kmax)
        took = "block_build" in B.sv_trace_report()
        B.sv_trace_enable(False)
        assert took == (blocks and kmax == 0)
        out.append(s.tensor.clone())
    eps = 2.0 ** -53 if dt == "c128" else 2.0 ** -24
    assert torch.linalg.vector_norm(out[0] - out[1]).item() <= 16 * len(gates) * eps
    s.close()
