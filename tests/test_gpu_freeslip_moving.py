"""Spheres cut by free-slip faces that move along them: a face cell's
reflection is decided by the map the populations were streamed with, not by
the map of the level they are gathered for."""
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


@pytest.mark.parametrize("dynamic", [False, True])
@pytest.mark.parametrize("faces", ["x-", "y+", "z-", "z both", "edge", "corner"])
def test_sphere_sliding_along_a_free_slip_face(lb, oracle_mod, faces, dynamic):
    """FP64 fields, maps and forces of every step against the oracle (the
    operations are the oracle's, so only the order of the sums differs)."""
    shape = (21, 18, 20)
    per, slip, X, U = {
        "x-": ((False, True, True), (1, 0, 0, 0, 0, 0), [(1.2, 9.3, 10.1)], [(0.02, 0.37, -0.23)]),
        "y+": ((True, False, True), (0, 0, 0, 1, 0, 0), [(9.0, 16.6, 10.1)], [(-0.41, 0.03, 0.3)]),
        "z-": ((True, True, False), (0, 0, 0, 0, 1, 0), [(9.0, 8.1, 0.3)], [(0.33, 0.29, 0.0)]),
        "z both": ((True, True, False), (0, 0, 0, 0, 1, 1), [(5.0, 8.1, 1.4), (15.2, 9.0, 18.9)],
                   [(0.33, 0.29, 0.0), (-0.2, 0.41, 0.05)]),
        "edge": ((False, False, True), (1, 1, 1, 0, 0, 0), [(2.0, 1.5, 9.9)], [(0.3, -0.1, 0.38)]),
        "corner": ((False, False, False), (1, 1, 1, 1, 1, 1), [(2.0, 1.5, 17.8), (13.0, 16.1, 2.2)],
                   [(0.3, 0.24, -0.28), (0.1, -0.3, 0.0)]),
    }[faces]
    X, U = np.array(X), np.array(U)
    n = len(X)
    R = np.array([3.6, 4.2])[:n]
    W = np.full((n, 3), 3e-3)
    rng = np.random.default_rng(3)
    N = shape[0] * shape[1] * shape[2]
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    f0 = w[:, None] * (1.0 + 0.01 * rng.uniform(-1, 1, (19, N)))
    o = oracle_mod.Oracle(shape, per)
    g = lb.Lattice(shape, per, precision=lb.FP64, move_particles=True)
    for t in (o, g):
        t.set_free_slip(slip)
        t.set_pdfs(f0)
    o.set_particles(X, R, U, W, moving=True)
    g.set_particles(X, R, U, W)
    if dynamic:
        for t in (o, g):
            t.set_dynamics(60.0, np.full(n, 0.1), (1e-3, 2e-3, 0.0))
    for k in range(9):
        o.step(1)
        g.step(1)
        fo, oo = o.map()
        fg, og = g.map()
        assert (fg == fo).all() and (og == oo).all(), k
        Fo, Mo = o.ft()
        Fg, Mg = g.ft()
        s = max(np.abs(Fo).max(), 1e-6)
        assert np.abs(Fg - Fo).max() <= 1e-12 * s, k
        assert np.abs(Mg - Mo).max() <= 1e-11 * s * R.max(), k
        if k % 2 == 0:  # the other steps gather in the sweep, not in a read-out
            _, u_o = o.macro()
            _, u_g = g.macro()
            assert np.abs(u_g - u_o).max() <= 1e-13, k
    # populations of the cells that were fluid all along
    fo, fg = o.get_pdfs(), g.get_pdfs()
    fluid = o.map()[0] % 3 == 0  # FLUID or NEAR
    assert np.abs(fg - fo)[:, fluid].max() <= 1e-13
    assert abs(g.invariants()[0] - o.invariants()[0]) <= 1e-11 * N
    g.close()
