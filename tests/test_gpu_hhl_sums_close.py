"""The fused complex64 solve against the unfused complex128 one, as close as its
roundings let it be: each of the three scalars is a mean of squares, whose single
roundings average out, so 64 roundings of the type cover solves of up to 2^23
amplitudes; x is a unit vector after two basis changes, 256 roundings.
"""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


@pytest.mark.parametrize("hi,lo,n_c", [(1, 0, 2), (2, 0, 3), (5, 0, 8), (10, 0, 4), (11, 0, 4), (6, 6, 9), (7, 6, 9)])
def test_fused_scalars_are_close(hi, lo, n_c):
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
    res = {}
    for d, mode in (("c128", 2), ("c64", 1)):
        st = B.State(n_s + n_c + 1, d)
        plan = B.sv_hhl_prepare(st.h, A_hi, A_lo)
        res[d] = B.sv_hhl_run(plan, st.h, b, n_c, T0, mode)
        B.sv_hhl_plan_free(plan)
        st.close()
    x2, r2 = res["c128"]
    x1, r1 = res["c64"]
    assert np.linalg.norm(x1 - x2) <= 256 * EPS
    for k in ("p_post", "p_anc", "norm_total"):
        assert abs(getattr(r1, k) - getattr(r2, k)) <= 64 * EPS * abs(getattr(r2, k)), (k, getattr(r1, k) / getattr(r2, k) - 1)
