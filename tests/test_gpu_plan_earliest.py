"""sv_apply_circuit with passes planned from the earliest gates (a fourth value 1
in the tuning entry of a circuit), against numpy, and the entry without it.
Tolerance: a rounding per gate and amplitude on a unit state.
"""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu

EPS = {"c128": 2.0 ** -53, "c64": 2.0 ** -24}


@pytest.mark.parametrize("dt,k,c,rb", [("c64", 13, 4, 5), ("c64", 12, 5, 4), ("c128", 12, 4, 4)])
def test_earliest_gate_passes(dt, k, c, rb):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, rng = 22, np.random.default_rng(k + c + rb)
    gates = []
    for _ in range(40):
        q = [int(x) for x in rng.choice(n, 2, replace=False)]
        gates.append(("u", q[0], inputs.random_unitary(rng, 2)) if rng.random() < 0.5 else
                     ("u", q[0], inputs.random_unitary(rng, 2), [q[1]], [1]))
    psi = inputs.random_state(rng, n)
    psi = psi.astype(np.complex64 if dt == "c64" else np.complex128).astype(np.complex128)
    ref = psi.copy()
    for g in gates:
        v = np.moveaxis(ref.reshape([2] * n), n - 1 - g[1], 0).copy()
        w = np.tensordot(g[2], v, axes=(1, 0))
        if len(g) > 3:
            ax = n - 1 - g[3][0]
            ax = ax + 1 if ax < n - 1 - g[1] else ax
            keep = [slice(None)] * n
            keep[ax] = 0
            w[tuple(keep)] = v[tuple(keep)]
        ref = np.ascontiguousarray(np.moveaxis(w, 0, n - 1 - g[1])).reshape(-1)
    s = B.State(n, dt)
    try:
        before = {ln.split()[0] for ln in B.sv_tune_report().splitlines()}
        s.set(psi)
        B.sv_apply_circuit(s.h, gates, 0)
        key = [ln.split()[0] for ln in B.sv_tune_report().splitlines()
               if ln.startswith(f"fused/{dt}/{n}/") and ln.split()[0] not in before]
        assert len(key) == 1
        for entry in ([k, c, rb, 1], [k, c, rb]):
            B.sv_tune_set(key[0], entry)
            s.set(psi)
            B.sv_apply_circuit(s.h, gates, 0)
            assert np.linalg.norm(s.get() - ref) <= 4 * len(gates) * EPS[dt], entry
        B.sv_tune_set(key[0], [])
    finally:
        s.close()
