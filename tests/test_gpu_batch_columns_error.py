"""complex64 batches are as accurate as they were when every solve ran as column
tiles: rms error of the four results over 1152 solves, relative to complex128, at
the clock widths where the columns were once worse.  The bounds are the column
tiles' errors on the same problems against 64 bits."""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu


def _problems(seed, n_c):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(24):
        n_s = int(rng.integers(3, 9))
        rng.integers(n_c, n_c + 1)
        A, _, lmax = inputs.random_spd_tridiag(rng, 1 << n_s, float(10.0 ** rng.uniform(1.0, 4.0)))
        out.append((A, rng.standard_normal(1 << n_s), n_c, inputs.t0_grid(lmax, 16)))
    return out


@pytest.mark.parametrize("n_c,bounds", [(8, (2.20e-7, 1.45e-7, 7.75e-8, 6.66e-8)), (9, (2.19e-7, 1.40e-7, 7.95e-8, 6.09e-8)),
                                        (10, (2.39e-7, 1.65e-7, 7.29e-8, 6.18e-8))])
def test_rms_errors(n_c, bounds, monkeypatch):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("SV_BATCH_QUEUE", "0")
    e = []
    for seed in range(3):
        p = _problems(seed, n_c)
        e.append(B.sv_hhl_batch(p, "c64") / B.sv_hhl_batch(p, "c128") - 1.0)
    rms = np.sqrt((np.concatenate(e) ** 2).mean(0))
    assert (rms <= np.array(bounds)).all(), rms
