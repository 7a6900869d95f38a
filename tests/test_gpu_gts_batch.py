"""Global steps queued in batches between status reads: the same states, times
and statistics as one step per call and as eager launches, also when the
target is reached inside a batch and when the run is called again after it."""
import numpy as np
import pytest

from workloads import concat_instances, sod_case, vortex_case

pytestmark = pytest.mark.gpu

KEYS = ("element_updates", "cycles", "macro_steps", "cfl_overshoots", "predictor_evals", "patches", "node_moves",
        "extra_cycles", "long_macro_steps", "t", "delta", "max_gcl_residual")


def _solver(M, instances):
    from paper_1408_3719_amd import Config, Solver

    if not instances:
        mesh, Q = vortex_case(500, seed=4)
        return Solver(mesh.nodes, mesh.tris, mesh.bedges, Q, Config(M=M))
    cases = [vortex_case(400 + 150 * k, seed=k) for k in range(3)]
    nodes, tris, bedges, Q, first = concat_instances(cases)
    return Solver(nodes, tris, bedges, Q, Config(M=M), instance_first=first)


def _state(s, st):
    Q, X, t = s.download()
    return Q, X, t, s.instance_times(), tuple(st[k] for k in KEYS)


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a[:4], b[:4])) and a[4] == b[4]


@pytest.mark.parametrize("instances", [False, True])
@pytest.mark.parametrize("steps", [1, 7, 8, 9, 21])
def test_batched_steps_equal_single_steps(steps, instances):
    a, b, c = (_solver(2, instances) for _ in range(3))
    c.set_graphs(False)
    st_a = a.step_gts(1e9, steps)
    for _ in range(steps):
        st_b = b.step_gts(1e9, 1)
    st_c = c.step_gts(1e9, steps)
    one = _state(a, st_a)
    assert st_a["macro_steps"] == steps
    assert _same(one, _state(b, st_b)) and _same(one, _state(c, st_c))


@pytest.mark.parametrize("instances", [False, True])
@pytest.mark.parametrize("n", [0.4, 2.5, 10.3, 17.0])
def test_target_inside_a_batch(n, instances):
    a, c = _solver(1, instances), _solver(1, instances)
    c.set_graphs(False)
    dt = float(a.dump("DTCFL").min())
    for k in (1, 2):   # the second call starts from the last report of the first
        st_a, st_c = a.step_gts(k * n * dt), c.step_gts(k * n * dt)
        assert _same(_state(a, st_a), _state(c, st_c))
        assert abs(st_a["t"] - k * n * dt) <= 1e-12 * max(1.0, k * n * dt)
    st = a.step_gts(2 * n * dt)   # already there: nothing to do
    assert st["macro_steps"] == st_a["macro_steps"] and st["t"] == st_a["t"]


def test_error_inside_a_batch_is_reported():
    from paper_1408_3719_amd import Config, Solver
    from paper_1408_3719_amd._lib import AderError

    mesh, Q = sod_case(600, seed=1408)
    s = Solver(mesh.nodes, mesh.tris, mesh.bedges, Q, Config(M=1))
    with pytest.raises(AderError):   # the unlimited scheme breaks down on so coarse a tube
        s.step_gts(0.2)
    with pytest.raises(AderError):   # the error stays until the next upload
        s.step_gts(0.2)
    s.upload_state(Q)
    assert s.step_gts(1e9, 1)["macro_steps"] == 1
