"""Fused solves whose column tiles are narrower than the tuner's candidates have
more tiles, and so more partial sums: the default without tuning of complex128
on a 20-qubit clock (4 columns), and pinned tiles of 1, 2 and 4 columns.  The
unfused solve of the same plan is the reference; both round every amplitude a
few hundred times at unit scale, and no error grows with the clock since both
read the same phases.
"""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"c128": 1e-12, "c64": 2e-5}


@pytest.mark.parametrize("dt,n_s,n_c,cl", [("c128", 3, 20, None), ("c128", 4, 19, None), ("c128", 5, 6, 0), ("c128", 5, 6, 1),
                                           ("c64", 5, 6, 0), ("c64", 6, 5, 2)])
def test_narrow_tiles_match_the_unfused_solve(dt, n_s, n_c, cl, monkeypatch):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(10 * n_s + n_c)
    A, _, lmax = inputs.random_spd_tridiag(rng, 1 << n_s, 20.0)
    b = rng.standard_normal(1 << n_s)
    T0 = inputs.t0_top_of_clock(lmax, n_c)
    key = f"eigpipe/{dt}/{n_s}/{n_c}"
    monkeypatch.setenv("SV_AUTOTUNE", "0")
    B.sv_tune_set(key, [] if cl is None else [cl, 256, cl, 256, 0, 0])
    st = B.State(n_s + n_c + 1, dt)
    plan = B.sv_hhl_prepare(st.h, A)
    try:
        x2, r2 = B.sv_hhl_run(plan, st.h, b, n_c, T0, 2)
        x1, r1 = B.sv_hhl_run(plan, st.h, b, n_c, T0, 1)
    finally:
        B.sv_hhl_plan_free(plan)
        st.close()
        B.sv_tune_set(key, [])
    assert np.linalg.norm(x1 - x2) <= TOL[dt]
    for k in ("p_post", "p_anc", "norm_total"):
        assert abs(getattr(r1, k) - getattr(r2, k)) <= TOL[dt] * abs(getattr(r2, k)), k
