"""Times, tick lengths and statistics that the host reports are those of the
device at the call, whatever ran since the last report."""
import numpy as np
import pytest

from workloads import concat_instances, sod_case, vortex_case

pytestmark = pytest.mark.gpu


def _solver(M=2, levels=3, n=500):
    from paper_1408_3719_amd import Config, Solver

    mesh, Q = vortex_case(n, seed=4)
    return Solver(mesh.nodes, mesh.tris, mesh.bedges, Q, Config(M=M, levels=levels)), mesh, Q


@pytest.mark.parametrize("keep", [-1, 1, 0])
def test_instance_times_after_an_lts_adjoint(keep):
    """Replayed macro steps report their own times before the end state comes back."""
    s, mesh, Q = _solver()
    a, _, _ = _solver()
    end = a.step_lts(1e9, 3)["t"]
    rng = np.random.default_rng(1)
    _, _, done = s.adjoint_lts(3, 1e9, rng.standard_normal(Q.shape), rng.standard_normal(mesh.nodes.shape), keep=keep)
    assert done == 3
    assert s.instance_times()[0] == end   # before any other call reads the status
    assert s.stats()["t"] == end


def test_instance_times_after_an_injected_time():
    s, _, _ = _solver()
    s.step_lts(1e9, 1)
    v = s.dump("SCAL")
    v[0] = 0.625
    s.inject("SCAL", v)
    assert s.instance_times()[0] == 0.625


@pytest.mark.parametrize("levels", [1, 3, 0])
def test_a_run_without_a_step_still_synchronises(levels):
    """The caller's work queued before the call is done when it returns."""
    import torch

    s, _, _ = _solver(levels=levels)
    step = s.step_gts if levels == 1 else s.step_lts
    t = step(0.05)["t"]
    a = torch.ones(4096, 4096, dtype=torch.float64, device=s.device)
    for _ in range(3):
        a @ a                     # the library's first calls
    torch.cuda.synchronize()
    for _ in range(40):           # ~80 ms
        b = a @ a
    assert not s.stream.query()
    step(t)
    assert s.stream.query()
    assert float(b[0, 0]) == 4096.0


@pytest.mark.parametrize("levels", [1, 3])
def test_a_macro_step_begun_again_takes_the_steps_as_they_are(levels):
    """The tick length follows the CFL steps at the begin, larger ones too."""
    s, _, _ = _solver(levels=levels)
    s.debug_macro_begin(1e9, levels)
    first = s.dump("SCAL")[1]
    s.inject("DTCFL", 4.0 * s.dump("DTCFL"))
    s.debug_macro_begin(1e9, levels)
    assert s.dump("SCAL")[1] == 4.0 * first
    a, _, _ = _solver(levels=levels)
    a.inject("DTCFL", 4.0 * a.dump("DTCFL"))
    a.debug_macro_begin(1e9, levels)
    assert np.array_equal(a.dump("STEP"), s.dump("STEP"))


@pytest.mark.parametrize("levels", [1, 3])
def test_a_macro_step_begun_at_its_target_stands_still(levels):
    """No instance is open: every element stays at the time reached."""
    s, _, _ = _solver(levels=levels)
    step = s.step_gts if levels == 1 else s.step_lts
    t = step(0.05)["t"]
    s.debug_macro_begin(t, levels)
    assert s.dump("SCAL")[1] == 0.0
    assert (s.download()[2] == t).all()


def _failing(batch):
    """A tube too coarse for the unlimited scheme, alone or between two vortices."""
    from paper_1408_3719_amd import Config, Solver

    mesh, Q = sod_case(600, seed=1408)
    if not batch:
        return Solver(mesh.nodes, mesh.tris, mesh.bedges, Q, Config(M=1))
    nodes, tris, bedges, Q, first = concat_instances([vortex_case(300, seed=1), (mesh, Q), vortex_case(400, seed=2)])
    return Solver(nodes, tris, bedges, Q, Config(M=1), instance_first=first)


def _after(s):
    """State, steps, times and statistics, whatever they hold."""
    st = s.stats()
    return [*s.download(), s.instance_times(), s.dump("TICK"), s.dump("STEP"), s.dump("NTICK"), s.dump("WNOD"),
            s.dump("DTCFL"), s.dump("SCAL"), np.array([float(st[k]) for k in st])]


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("before", [0, 3, 6])
def test_a_failed_run_stops_at_the_step_that_failed(batch, before):
    """Steps queued behind it leave everything as eager launches do, which
    stop there; `before` single steps move it inside the queue."""
    from paper_1408_3719_amd import AderError

    a, b = _failing(batch), _failing(batch)
    b.set_graphs(False)
    for s in (a, b):
        for _ in range(before):
            s.step_gts(1e9, 1)
        with pytest.raises(AderError):
            s.step_gts(2.0)
    assert a.stats()["macro_steps"] == b.stats()["macro_steps"] > before
    for x, y in zip(_after(a), _after(b)):
        assert np.array_equal(x, y, equal_nan=True)


def test_steps_after_another_workspace_is_bound():
    """The captured steps are those of the workspace that is bound (the one
    before stays allocated here)."""
    import ctypes

    import torch

    s, _, Q = _solver(levels=1)
    s.step_gts(1e9, 5)
    want = s.download()
    n = ctypes.c_size_t()
    assert s.lib.ader_workspace_size(s.ctx, ctypes.byref(n)) == 0
    other = torch.empty(n.value + 256, dtype=torch.uint8, device=s.device)
    at = (other.data_ptr() + 255) // 256 * 256
    assert s.lib.ader_bind_workspace(s.ctx, ctypes.c_void_p(at), n.value) == 0
    s.upload_state(Q)
    s.step_gts(1e9, 5)
    for a, b in zip(s.download(), want):
        assert np.array_equal(a, b)
    s.close()
