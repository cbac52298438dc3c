"""The read-out that gathers from the post-collision state: the same values as
from the post-stream state in the grid, and no change of the state."""
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


@pytest.mark.parametrize("faces", ["ppp", "fnf", "wpf"])
@pytest.mark.parametrize("force", ["dense", "charge", "psi"])
@pytest.mark.parametrize("prec", ["FP64", "FP32DEV", "FP16DEV"])
def test_readout_gathers_what_the_next_step_will(lb, prec, force, faces):
    """Bitwise: the gather moves stored values, and a refill is rounded to the
    storage format either way."""
    shape = (38, 30, 26)
    N = 38 * 30 * 26
    per = tuple(f == "p" for f in faces)
    rng = np.random.default_rng(3)
    field = rng.uniform(0.5, 1.0, 3 * N) * 1e-4
    # FP16 holds deviations below 2^-6: surface velocities to match
    U = np.array([[0.11, -0.07, 0.05], [-0.09, 0.1, 0.02]]) * (0.05 if prec == "FP16DEV" else 1.0)
    fl = np.zeros(shape[::-1], dtype=np.uint8)
    if faces[0] == "w":
        fl[:, :, 0] = fl[:, :, -1] = 1

    def lattice():
        L = lb.Lattice(shape, per, precision=getattr(lb, prec), move_particles=True)
        L.set_flags(fl)
        if "f" in faces:
            L.set_free_slip([f == "f" for f in faces for _ in range(2)])
        L.init_equilibrium(1.0, (1e-3, 2e-3, -1e-3))
        L.set_particles(np.array([[12.0, 11.3, 12.9], [26.2, 18.0, 13.5]]), np.array([4.0, 3.1]),
                        U, np.full((2, 3), 1e-3))
        if force == "dense":
            L.set_force(field)
        elif force == "charge":
            L.set_charge_force(field[:N], (1.0, -0.5, 0.3))
        else:
            L.set_potential_force(field[:N], 0.1, (1.0, -0.5, 0.3), np.array([0.02, -0.03]))
        return L

    a, b = lattice(), lattice()
    for k in (1, 2, 9):
        a.step(k)
        b.step(k)
        rho, u = a.macro()   # gathers
        again = a.macro()
        pdfs = b.get_pdfs()  # brings b to its post-stream state
        ref = b.macro()
        assert np.isfinite(pdfs).all()
        assert (rho == ref[0]).all() and (u == ref[1]).all()
        assert (again[0] == rho).all() and (again[1] == u).all()
    assert (a.get_pdfs() == pdfs).all()
    a.close()
    b.close()
