"""Device memory that one LTS adjoint leaves with its context for the next:
calls of different sizes on one context give the bits that a fresh context
gives."""
import numpy as np
import pytest

from workloads import vortex_case

pytestmark = pytest.mark.gpu


def _solver(case):
    from paper_1408_3719_amd import Config, Solver

    mesh, Q = case
    return Solver(mesh.nodes, mesh.tris, mesh.bedges, Q, Config(M=2, levels=3))


def _gradient(s, case, n, keep, seed):
    mesh, Q = case
    rng = np.random.default_rng(seed)
    s.upload_state(Q)
    gq, gx, done = s.adjoint_lts(n, 1e9, rng.standard_normal(Q.shape), rng.standard_normal(mesh.nodes.shape), keep=keep)
    assert done == n
    return gq.cpu().numpy(), gx.cpu().numpy()


def test_calls_of_different_sizes_on_one_context():
    case = vortex_case(900, seed=3)
    s = _solver(case)
    for n, keep, seed in ((2, -1, 1), (1, -1, 2), (4, -1, 3), (3, 1, 4), (3, 0, 5), (14, -1, 6), (2, -1, 1)):
        a = _gradient(s, case, n, keep, seed)
        f = _solver(case)
        b = _gradient(f, case, n, keep, seed)
        f.close()
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), (n, keep)
    # a call that fails gives its blocks back; the next one is as before
    from paper_1408_3719_amd import AderError

    mesh, Q = case
    bad = Q.copy()
    bad[mesh.n_elems // 2, 0] = -1.0
    with pytest.raises(AderError):
        s.upload_state(bad)
        s.adjoint_lts(2, 1e9, Q, mesh.nodes)
    c = _gradient(s, case, 2, -1, 1)
    assert np.array_equal(a[0], c[0]) and np.array_equal(a[1], c[1])
