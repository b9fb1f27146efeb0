"""The matrix-core product with its k range in parts (tile shapes 2 and 3 of
the cgemm tuning entry), at the edges of its tiles and chunks: fewer rows than a
tile, k shorter than one chunk of every part, registers off the bottom of the
state, adjoints, and the largest shape the parts are picked for.  Against numpy;
tolerance: K products and sums per entry, each within a rounding, of unit rows.
"""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu

EPS = {"c128": 2.0 ** -53, "c64": 2.0 ** -24}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("shape", [2, 3])
@pytest.mark.parametrize("n,lo,m,ctrl,adj", [
    (2, 0, 1, 1, 0), (5, 0, 4, -1, 1), (6, 0, 5, 5, 0), (9, 0, 4, 8, 1), (10, 2, 5, 9, 0), (11, 3, 6, 1, 1),
    (13, 0, 7, 12, 1), (14, 0, 8, 13, 0), (15, 5, 8, 2, 0), (19, 0, 8, 18, 1), (18, 0, 9, -1, 0)])
def test_parts_match_dense_product(dt, shape, n, lo, m, ctrl, adj):
    import torch
    N = 1 << m
    rng = np.random.default_rng(31 * n + 7 * lo + m)
    U = inputs.random_unitary(rng, N)
    psi = inputs.random_state(rng, n)
    cd = np.complex128 if dt == "c128" else np.complex64
    U, psi = U.astype(cd), psi.astype(cd)
    rows = 1 << (n - m - (1 if ctrl >= 0 else 0))
    key = f"cgemm/{dt}/{rows}/{N}/{N}/{adj}" + (f"/s{lo}" if lo else "")
    s = B.State(n, dt)
    s.set(psi)
    B.sv_tune_set(key, [shape])
    try:
        Ud = torch.from_numpy(np.ascontiguousarray(U)).cuda()
        B.sv_apply_ctrl_unitary(s.h, Ud, lo, m, ctrl, 1, bool(adj))
        got = s.get()
    finally:
        B.sv_tune_set(key, [])
        s.close()
    W = U.astype(np.complex128)
    W = W.conj().T if adj else W
    v = psi.astype(np.complex128).reshape(-1, N, 1 << lo)
    ref = np.einsum("ab,xby->xay", W, v).reshape(-1)
    if ctrl >= 0:
        keep = (np.arange(1 << n) >> ctrl & 1) == 0
        ref[keep] = psi[keep]
        assert np.array_equal(got[keep], psi[keep].astype(np.complex128))
    assert np.linalg.norm(got - ref) <= 4 * np.sqrt(N) * EPS[dt] * np.linalg.norm(ref)
