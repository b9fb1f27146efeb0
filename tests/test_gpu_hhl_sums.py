"""The fused solve's sums and vector steps where their launches change: one or 64
stretches of partial sums (register sizes 22 and 23), one or 64 workgroups for
|b| and |x| (4096 and 8192 unknowns), one or two row segments of a dense basis
(1024 and 2048 unknowns) and the smallest systems.  The unfused solve of the
same plan is the reference; tolerance: both round every amplitude a few hundred
times at unit scale.
"""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"c128": 1e-12, "c64": 2e-4}


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("hi,lo,n_c", [(1, 0, 2), (1, 1, 2), (2, 0, 3), (10, 0, 4), (11, 0, 4), (6, 6, 9), (7, 6, 9)])
def test_fused_sums_match_the_unfused_solve(dt, hi, lo, n_c):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(100 * hi + lo)
    if lo:
        ks = inputs.kron_laplacian_system(rng, hi, lo, kappa=20.0)
        A_hi, A_lo, lmax = ks.A_hi, ks.A_lo, ks.lambda_max
    else:
        A_hi, _, lmax = inputs.random_spd_tridiag(rng, 1 << hi, 20.0)
        A_lo = None
    n_s = hi + lo
    T0 = inputs.t0_top_of_clock(lmax, n_c)
    b = rng.standard_normal(1 << n_s) + 1j * rng.standard_normal(1 << n_s)
    st = B.State(n_s + n_c + 1, dt)
    plan = B.sv_hhl_prepare(st.h, A_hi, A_lo)
    try:
        x2, r2 = B.sv_hhl_run(plan, st.h, b, n_c, T0, 2)
        x1, r1 = B.sv_hhl_run(plan, st.h, b, n_c, T0, 1)
        b_dev = torch.tensor(b, device="cuda")
        x_dev = torch.empty(1 << n_s, dtype=torch.complex128, device="cuda")
        rd = B.sv_hhl_run_device(plan, st.h, b_dev, n_c, T0, 1, x_dev=x_dev)
        xd = x_dev.cpu().numpy()
    finally:
        B.sv_hhl_plan_free(plan)
        st.close()
    for x, r in ((x1, r1), (xd, rd)):
        assert np.linalg.norm(x - x2) <= TOL[dt]
        for k in ("p_post", "p_anc", "norm_total"):
            assert abs(getattr(r, k) - getattr(r2, k)) <= TOL[dt] * abs(getattr(r2, k)), k
