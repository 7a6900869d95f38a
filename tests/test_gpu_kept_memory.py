"""Device memory that LTS adjoints leave with their contexts: bounded over all
contexts of the process, given back on request and by a call that fails."""
import numpy as np
import pytest

from workloads import explosion_case, sod_case

pytestmark = pytest.mark.gpu


def _solver(case, M=2):
    from paper_1408_3719_amd import Config, Solver

    mesh, Q = case
    return Solver(mesh.nodes, mesh.tris, mesh.bedges, Q, Config(M=M, levels=3))


def _gradient(s, case, n):
    mesh, Q = case
    rng = np.random.default_rng(2)
    s.upload_state(Q)
    gq, gx, done = s.adjoint_lts(n, 1e9, rng.standard_normal(Q.shape), rng.standard_normal(mesh.nodes.shape))
    assert done == n
    return gq.cpu().numpy(), gx.cpu().numpy()


def _free(torch):
    """Free memory of the device but for what torch holds for itself."""
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()


def test_all_contexts_together_stay_within_the_bound():
    """Six contexts that would each keep ~3.6 GB."""
    import torch

    case = explosion_case(50_000, seed=1)
    a = [_solver(case) for _ in range(6)]
    total = torch.cuda.mem_get_info()[1]
    before = _free(torch)
    want = [_gradient(s, case, 8) for s in a]
    kept = before - _free(torch)
    slack = 256 << 20   # torch's own libraries
    print(f"kept {kept / 2**30:.2f} GiB of {total / 2**30:.1f}", flush=True)
    assert (1 << 30) < kept <= total // 16 + slack
    for s in a:
        s.release_memory()
    assert before - _free(torch) <= slack
    for s, w in zip(a, want):   # as before, and the room is there again
        g = _gradient(s, case, 8)
        assert np.array_equal(g[0], w[0]) and np.array_equal(g[1], w[1])
    assert before - _free(torch) > (1 << 30)
    for s in a:
        s.close()
    assert _free(torch) >= before - slack


def test_a_gradient_that_fails_gives_its_memory_back():
    """The forward run of a tube too coarse for the scheme breaks down after the
    call has taken its memory; the next call is as on a fresh context."""
    import torch

    from paper_1408_3719_amd import AderError

    case = sod_case(600, seed=1408)
    mesh, Q = case
    s, fresh = _solver(case, M=1), _solver(case, M=1)
    want = _gradient(fresh, case, 3)
    before = _free(torch)
    _gradient(s, case, 3)
    s.upload_state(Q)
    with pytest.raises(AderError):
        s.adjoint_lts(1000, 1e9, Q, mesh.nodes)
    assert s.stats()["macro_steps"] > 3   # inside the forward run
    assert before - _free(torch) <= 2 << 20
    got = _gradient(s, case, 3)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
