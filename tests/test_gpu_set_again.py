"""A new particle table after any number of steps: the maps of a lattice that
has seen only that table (the next level's map is taken as the steps left it)."""
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


@pytest.mark.parametrize("free", [False, True])
@pytest.mark.parametrize("first", [0, 1, 2, 3, 4])
def test_maps_after_a_new_table(lb, first, free):
    rng = np.random.default_rng(5)
    shape = (33, 30, 27)

    def table(n, R):
        return rng.random((n, 3)) * np.array(shape), np.full(n, R), rng.uniform(-0.4, 0.4, (n, 3))
    old, new = table(9, 5.2), table(14, 3.3)
    g = lb.Lattice(shape, precision=lb.FP32DEV, move_particles=True)
    for k, t in enumerate((old, new, (np.zeros((0, 3)), np.zeros(0), np.zeros((0, 3))), new, old)):
        g.set_particles(*t)
        if len(t[1]) == 0:
            g.step(first)
            assert (g.map()[1] == -1).all()
            continue
        h = lb.Lattice(shape, precision=lb.FP32DEV, move_particles=True)
        h.set_particles(*t)
        if free and k == 0:
            g.set_dynamics(1e9)  # too heavy to change its velocity in the maps
        for s in range(first + 1):
            for a, b in zip(g.map(), h.map()):
                assert (a == b).all(), (k, s)
            g.step(1)
            h.step(1)
        h.close()
    g.close()
