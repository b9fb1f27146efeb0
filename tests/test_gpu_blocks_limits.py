"""Pinned configurations that the matrix-core blocks cannot run are refused on
the host, before anything is launched, and leave the state as it is."""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("k,wide", [(14, False), (7, False), (12, True)])
def test_pinned_blocks_out_of_range_are_refused(dt, k, wide):
    """A tile of 14 or 7 qubits; a gate of five qubits."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 22
    rng = np.random.default_rng(40 + k)
    gates = inputs.random_circuit(rng, n, 12)
    if wide:
        gates.append(("u", 3, inputs.random_unitary(rng, 2), [0, 9, 12, 21], [1, 0, 1, 1]))
    s = B.State(n, dt)
    B.sv_init_basis(s.h, 5)
    before = set(B.sv_tune_report().splitlines())
    B.sv_apply_circuit(s.h, gates)
    key, = [ln.split()[0] for ln in B.sv_tune_report().splitlines() if ln.startswith("fused/") and ln not in before]
    psi = s.tensor.clone()
    try:
        B.sv_tune_set(key, [k, 3, 1])
        with pytest.raises(B.SvError) as e:
            B.sv_apply_circuit(s.h, gates)
        assert e.value.status == B.SV_EINVAL
        assert torch.equal(s.tensor, psi)
    finally:
        B.sv_tune_set(key, [])
        s.close()
