"""Global steps list the unfinished elements without a look at their stencils;
the same steps replayed from a schedule go through the update criterion. Both
give the same states, as do all chunk sizes of the criterion's scan."""
import numpy as np
import pytest

from workloads import vortex_case

pytestmark = pytest.mark.gpu


def _solver(n):
    from paper_1408_3719_amd import Config, Solver

    mesh, Q = vortex_case(n, seed=n)
    return Solver(mesh.nodes, mesh.tris, mesh.bedges, Q, Config(M=1, levels=3))


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a.download(), b.download()))


# below, around and well above a chunk of 1024 elements
@pytest.mark.parametrize("n", [60, 1000, 1100, 2100, 5000])
def test_global_steps_equal_their_replay(n):
    a, b = _solver(n), _solver(n)
    a.record_schedule(8, 8)
    st_a = a.step_gts(1e9, 3)
    log, _ = a.recorded_schedule()
    assert all(len(x) == 3 for x in log)
    b.set_schedule_replay(log)
    st_b = b.step_gts(1e9, 3)
    assert st_a["element_updates"] == st_b["element_updates"] == 3 * a.NE
    assert _same(a, b)


@pytest.mark.parametrize("n", [1100, 40000])
@pytest.mark.parametrize("chunk", [128, 1000, 1024])
def test_chunk_size_does_not_change_the_steps(n, chunk):
    a, b = _solver(n), _solver(n)
    b.set_tune(sched_chunk=chunk)
    st_a, st_b = a.step_lts(1e9, 2), b.step_lts(1e9, 2)
    assert st_a["element_updates"] == st_b["element_updates"] and st_a["cycles"] == st_b["cycles"]
    assert _same(a, b)
