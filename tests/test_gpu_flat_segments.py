"""The sweep's flat segments (consecutive cells across rows and planes) at the
extents where a lane's place is derived differently: rows of one cell, rows
shorter and longer than a segment, both sides of 2048 along x and y, with
periodic and bounce-back edges, in both sweep modes and the read-out."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    assert torch.cuda.is_available()
    from paper_1708_08741_amd import lbmep
    lbmep.lib()
    return lbmep


@pytest.mark.parametrize("per", [(True, True, True), (False, True, False), (False, False, False)])
@pytest.mark.parametrize("shape", [(1, 5, 7), (5, 1, 9), (1, 1, 300), (2, 3, 43), (63, 5, 3),
                                   (65, 3, 3), (129, 2, 2), (2047, 3, 2), (2048, 1, 3),
                                   (2049, 2, 1), (2, 2047, 2), (1, 2050, 1), (4099, 1, 1)])
def test_flat_segments_against_the_oracle(lb, oracle_mod, shape, per):
    """FP64: the operations of the oracle on the same values, so equal up to
    its summation of the moments (1e-15 of values of order 1; bound 1e-13)."""
    rng = np.random.default_rng(5)
    N = shape[0] * shape[1] * shape[2]
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    f0 = w[:, None] * (1.0 + 0.01 * rng.uniform(-1, 1, (19, N)))
    fb = rng.uniform(-1e-4, 1e-4, (3, N))
    o = oracle_mod.Oracle(shape, per)
    g = lb.Lattice(shape, per, precision=lb.FP64)
    for t in (o, g):
        t.set_force(fb)
        t.set_pdfs(f0)
        t.step(4)
    assert np.abs(g.get_pdfs().reshape(19, N) - o.get_pdfs().reshape(19, N)).max() <= 1e-13
    g.close()
