"""A non-finite potential stays on its side of walls and spheres during a
solve: no form of the iteration reads a solid cell's value as a neighbour's."""
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


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("prec", ["FP32DEV", "FP64"])
@pytest.mark.parametrize("shape,axis,solid", [
    ((16, 20, 24), 0, "wall"), ((16, 20, 24), 1, "wall"), ((16, 20, 24), 2, "wall"),
    ((140, 12, 8), 0, "wall"), ((520, 12, 8), 0, "wall"), ((520, 12, 8), 1, "wall"),
    ((6, 6, 24), 2, "sphere"), ((24, 6, 6), 0, "sphere")])
def test_the_other_side_does_not_see_it(lb, monkeypatch, shape, axis, solid, prec, bad):
    """Bitwise the in-place half-sweeps' values beyond the solid cells."""
    import torch
    dtype = torch.float64 if prec == "FP64" else torch.float32
    nx, ny, nz = shape
    rng = np.random.default_rng(2)
    psi = rng.uniform(-1, 1, (nz, ny, nx))
    mid = shape[axis] // 2
    place = [slice(None)] * 3
    place[2 - axis] = mid
    put = [nz // 2, ny // 2, nx // 2]
    put[2 - axis] = mid - 4 if solid == "sphere" else mid - 1
    put = [max(v, 0) for v in put]
    if solid == "sphere":  # fills the cross-section
        put[2 - axis] = 1
    psi[tuple(put)] = bad
    out = []
    for fused in ("1", "0"):
        monkeypatch.setenv("LBMEP_SOR_FUSED", fused)
        L = lb.Lattice(shape, (False, False, False), precision=getattr(lb, prec))
        if solid == "wall":
            fl = np.zeros((nz, ny, nx), dtype=np.uint8)
            fl[tuple(place)] = 1
            L.set_flags(fl)
            zeta = None
        else:
            c = np.array([[0.5 * nx, 0.5 * ny, 0.5 * nz]])
            L.set_particles(c, np.array([5.0]), np.zeros((1, 3)))
            zeta = np.array([0.3])
        L.set_potential_force(torch.tensor(psi.reshape(-1), dtype=dtype, device="cuda"), 1e-3,
                              (0.0, 0.0, 0.0), zeta)
        L.set_potential_solver(0.05, 1.6, 41, 0.0, 1)
        L.solve_potential()
        out.append(L.potential().reshape(nz, ny, nx))
        L.close()
    beyond = [slice(None)] * 3
    beyond[2 - axis] = slice(mid + (3 if solid == "sphere" else 1), None)
    a, b = out[0][tuple(beyond)], out[1][tuple(beyond)]
    assert np.isfinite(b).all() and (a == b).all()
    # the solid cells keep their own values
    if solid == "wall":
        assert (out[0][tuple(place)] == out[1][tuple(place)]).all()
