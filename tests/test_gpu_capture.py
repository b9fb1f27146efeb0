"""Calls that stage host data refuse stream capture: a recorded copy would read
whatever a later call has staged by the time the graph is replayed."""
import numpy as np
import pytest

from paper_2307_00391_amd import binding as B
from paper_2307_00391_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("kmax", [0, 9])
def test_circuits_refuse_capture_and_run_on(dt, kmax):
    """Blocks (kmax = 0) and vector passes, with the staging buffer in place from
    an earlier call; the call after the capture gives the result of a fresh state."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 10
    gates = inputs.probe_layers(np.random.default_rng(3), n, 2)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = B.State(n, dt)
        B.sv_init_basis(s.h, 3)
        B.sv_apply_circuit(s.h, gates, kmax)
        want = s.tensor.clone()
        B.sv_init_basis(s.h, 3)
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        with pytest.raises(B.SvError) as e:
            B.sv_apply_circuit(s.h, gates, kmax)
        B.sv_qft(s.h, 0, n)           # a call that stages nothing is recorded
    assert e.value.status == B.SV_EUNSUPPORTED
    B.sv_apply_circuit(s.h, gates, kmax)
    stream.synchronize()
    assert torch.equal(s.tensor, want)
    s.close()


@pytest.mark.parametrize("mode", [0, 1])
def test_solves_from_the_host_refuse_capture_and_run_on(mode):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n_s, n_c = 3, 5
    rng = np.random.default_rng(4)
    A, _, lmax = inputs.random_spd_tridiag(rng, 1 << n_s, 20.0)
    b = rng.standard_normal(1 << n_s)
    T0 = inputs.t0_top_of_clock(lmax, n_c)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = B.State(n_s + n_c + 1, "c128")
        plan = B.sv_hhl_prepare(s.h, A)
        x0, _ = B.sv_hhl_run(plan, s.h, b, n_c, T0, mode)
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        with pytest.raises(B.SvError) as e:
            B.sv_hhl_run(plan, s.h, b, n_c, T0, mode)
        B.sv_qft(s.h, 0, n_s)
    assert e.value.status == B.SV_EUNSUPPORTED
    x1, _ = B.sv_hhl_run(plan, s.h, b, n_c, T0, mode)
    assert np.array_equal(x0, x1)
    B.sv_hhl_plan_free(plan)
    s.close()
