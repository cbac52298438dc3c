"""Free spheres whose velocity reaches one cell per step: the position stays
in the components that do, so the maps, marks and owners keep belonging
together and every later call has defined cells to work on."""
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


@pytest.mark.parametrize("prec", ["FP64", "FP32DEV"])
@pytest.mark.parametrize("E", [(3.0, 0.0, 0.0), (-1.0, 0.02, 40.0), (1e308, 0.0, 0.0)])
def test_a_component_of_one_cell_does_not_move_the_sphere(lb, E, prec):
    """The first step from rest gives U = q E / m with no exchange force: the
    components of E below 1 move the sphere by it, the others do not."""
    shape, R, rho_p = (26, 24, 22), 3.0, 1.5
    X = np.array([[8.0, 12.0, 11.0], [19.0, 12.0, 11.0]])
    m = rho_p * 4.0 / 3.0 * np.pi * R ** 3
    g = lb.Lattice(shape, precision=getattr(lb, prec), move_particles=True)
    g.set_particles(X, [R, R], np.zeros((2, 3)))
    g.set_potential_force(np.zeros(shape[::-1]), 1e-3, (0.0, 0.0, 0.0), [0.1, -0.1])
    g.set_potential_solver(0.05, 1.6, 4, 0.0, 1)
    g.set_dynamics(rho_p, [2.0 * m, 0.0], E)  # U = 2 E
    flags, owner = g.map()
    g.step(1)
    with pytest.raises(lb.LbmepError, match="one cell per step"):
        g.particles()
    slow = [a for a in range(3) if abs(2.0 * E[a]) < 1.0]
    if all(E[a] == 0.0 for a in slow):  # nothing has moved
        f1, o1 = g.map()
        assert (f1 == flags).all() and (o1 == owner).all()
    else:  # a way of 0.04 along y takes no cell centre into or out of the ball
        assert (g.map()[1] == owner).all()
    # the motion is not the body's any more; every entry point still runs
    for k in range(6):
        g.step(3)
        g.macro()
        g.get_pdfs()
        g.solve_potential()
        o = g.map()[1]
        assert ((o >= -1) & (o < 2)).all() and (o >= 0).sum() >= (owner >= 0).sum() // 2
    with pytest.raises(lb.LbmepError, match="one cell per step"):
        g.particles()
    # a new table starts anew
    g.set_particles(X, [R, R], np.zeros((2, 3)))
    assert (g.particles()[0] == X).all() and (g.map()[1] == owner).all()
    g.close()
