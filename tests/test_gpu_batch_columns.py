"""Batched solves, a column per lane (the form without work queues), at the edges
of its lines and splits: clock widths below a line (2..4), lines with no, one,
two and three root bits (5..8), the first with low bits, widths that split over
workgroups (13, 16), systems of one qubit (padded lanes) and one with a full
workgroup of columns.  Against single fused solves of the same problems.
Tolerance: relative, every amplitude within a few hundred roundings."""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu

REL = {"c128": 1e-11, "c64": 2e-5}


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("shapes", [[(1, 2), (1, 3), (2, 4)], [(1, 5), (3, 6), (2, 7), (6, 8)],
                                    [(5, 9), (1, 13), (2, 16)], [(7, 12)], [(1, 2), (8, 10), (1, 11)]])
def test_columns_match_single_solves(dt, shapes, monkeypatch):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("SV_BATCH_QUEUE", "0")
    rng = np.random.default_rng(sum(31 * a + b for a, b in shapes))
    probs = []
    for n_s, n_c in shapes:
        A, _, lmax = inputs.random_spd_tridiag(rng, 1 << n_s, 8.0)
        probs.append((A, rng.standard_normal(1 << n_s), n_c, inputs.t0_top_of_clock(lmax, n_c) * np.array([0.6, 0.9, 0.97])))
    res = B.sv_hhl_batch(probs, dt)
    k = 0
    for A, b, n_c, t0s in probs:
        n_s = A.shape[0].bit_length() - 1
        x = np.linalg.solve(A, b)
        st = B.State(n_s + n_c + 1, dt)
        try:
            for T0 in t0s:
                xq, r = B.sv_hhl(st.h, A, b, n_c, float(T0), 1)
                F = abs(np.vdot(x, xq)) / np.linalg.norm(x)
                assert abs(res[k, 0] - r.p_post) <= REL[dt] * r.p_post, (n_s, n_c, res[k, 0], r.p_post)
                assert abs(res[k, 1] - r.p_anc) <= REL[dt] * r.p_anc, (n_s, n_c)
                assert abs(res[k, 2] - r.norm_total) <= REL[dt]
                assert abs(res[k, 3] - F) <= REL[dt], (n_s, n_c, res[k, 3], F)
                k += 1
        finally:
            st.close()
