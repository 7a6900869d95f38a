"""Times, tick lengths and statistics that the host reports are those of the
device at the call, whatever ran since the last report."""
import numpy as np
import pytest

from workloads import vortex_case

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
