"""Spheres that lie on wall cells' neighbours when they are set and move off:
the cells they uncover next to a wall get its bounce-back."""
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


@pytest.mark.parametrize("order", ["flags first", "particles first"])
@pytest.mark.parametrize("case", ["plane", "scattered", "large sphere"])
def test_sphere_leaves_the_wall_it_was_set_on(lb, oracle_mod, case, order):
    rng = np.random.default_rng(17)
    shape, per = ((44, 40, 38) if case == "large sphere" else (37, 33, 29)), (True, False, True)
    fl = np.zeros(shape[::-1], dtype=np.uint8)
    fl[:, 0, :] = fl[:, -1, :] = 1
    if case == "plane":
        X, R = np.array([[12.0, 4.2, 9.0], [25.0, 28.1, 20.0]]), np.array([4.5, 4.1])
        U = np.array([[0.1, 0.4, -0.2], [0.0, -0.3, 0.1]])
    elif case == "large sphere":  # classified cell by cell
        X, R, U = np.array([[20.0, 12.0, 19.0]]), np.array([12.5]), np.array([[0.1, 0.35, 0.0]])
    else:
        fl[rng.random(shape[::-1]) < 0.01] = 1
        X = rng.random((9, 3)) * np.array(shape)
        R, U = np.full(9, 4.5), rng.uniform(-0.3, 0.3, (9, 3))
    W = np.full_like(U, 2e-3)
    o = oracle_mod.Oracle(shape, per)
    g = lb.Lattice(shape, per, precision=lb.FP64, move_particles=True)
    o.set_flags(fl)
    o.init_equilibrium(1.0, (1e-3, 0.0, -1e-3))
    o.set_particles(X, R, U, W, moving=True)
    if order == "flags first":
        g.set_flags(fl)
    g.init_equilibrium(1.0, (1e-3, 0.0, -1e-3))
    g.set_particles(X, R, U, W)
    if order == "particles first":
        g.set_flags(fl)
    for k in (1, 2, 9):
        o.step(k)
        g.step(k)
        fo, oo = o.map()
        fg, og = g.map()
        assert (fg == fo).all() and (og == oo).all()
        Fo, Mo = o.ft()
        Fg, Mg = g.ft()
        s = max(np.abs(Fo).max(), 1e-6)
        assert np.abs(Fg - Fo).max() <= 1e-12 * s
        assert np.abs(Mg - Mo).max() <= 1e-11 * s * R.max()
        rho_o, u_o = o.macro()
        rho_g, u_g = g.macro()
        assert np.abs(u_g - u_o).max() <= 1e-13
        assert np.abs(rho_g - rho_o).max() <= 1e-12
    g.close()
