"""Staged stencils of the reconstruction: element numberings whose workgroups
name few and many different elements (a round of 32 elements, halved rounds
down to the smallest) give the same reconstruction, bit for bit."""
import numpy as np
import pytest

from workloads import vortex_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 2, 3])
@pytest.mark.parametrize("n", [300, 5000, 18000])
@pytest.mark.parametrize("block", [1, 8])
def test_reconstruction_does_not_depend_on_the_element_order(M, n, block):
    """block = 1: elements numbered at random, 32 consecutive ones share no
    stencil; block = 8: runs of 8 neighbours in random order. Rows, their order
    and the arithmetic are the same, so are the results."""
    from paper_1408_3719_amd import Config, Solver

    mesh, Q0 = vortex_case(n, seed=3)
    rng = np.random.default_rng(11)
    NE = mesh.n_elems
    runs = [np.arange(b, min(NE, b + block)) for b in range(0, NE, block)]
    order = np.concatenate([runs[k] for k in rng.permutation(len(runs))])
    cfg = Config(M=M, levels=2)
    a = Solver(mesh.nodes, mesh.tris, mesh.bedges, Q0, cfg)
    b = Solver(mesh.nodes, mesh.tris[order], mesh.bedges, Q0[order], cfg)
    assert np.array_equal(a.dump("DTCFL")[order], b.dump("DTCFL"))
    assert np.array_equal(a.dump("WNOD")[:, :, order], b.dump("WNOD"))
