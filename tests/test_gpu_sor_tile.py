"""The tile pass of the red-black SOR solver (one or two iterations per
launch) against the in-place one-launch-per-colour form, bitwise: rows at the
edges of its lanes and wavefronts, row blocks at the edges of its workgroups,
ranges of planes that meet two row blocks, stops at a residual between pairs
of iterations, and the rows that are too long for it."""
import numpy as np
import pytest

from paper_1708_08741_amd import workloads as W

pytestmark = pytest.mark.gpu

KEPS = 1e-3


@pytest.fixture(scope="module")
def lb():
    import torch
    assert torch.cuda.is_available()
    from paper_1708_08741_amd import lbmep
    lbmep.lib()
    return lbmep


def _case(shape, periodic, seed):
    rng = np.random.default_rng(seed)
    nx, ny, nz = shape
    psi = rng.standard_normal((nz, ny, nx))
    fl = np.zeros((nz, ny, nx), dtype=np.uint8)
    fl[rng.random((nz, ny, nx)) < 0.01] = 1
    n = 6
    X = rng.random((n, 3)) * np.array(shape)
    R = np.full(n, min(2.3, 0.45 * min(shape)))
    return psi, fl, X, R, rng.uniform(-0.5, 0.5, n)


def _solve(lb, monkeypatch, fused, case, shape, periodic, precision, iters, rf, every, zeta, solids):
    psi, fl, X, R, zv = case
    monkeypatch.setenv("LBMEP_SOR_FUSED", fused)
    g = lb.Lattice(shape, periodic, precision=precision)
    if solids:
        g.set_flags(fl)
        g.set_particles(X, R, np.zeros((len(R), 3)))
    g.set_potential_force(psi, KEPS, (0.0, 0.0, 0.0), zv if zeta and solids else None)
    g.set_potential_solver(0.3, 1.7, iters, rf, every)
    out = (g.solve_potential(), g.potential(), g.solver_shape())
    g.close()
    return out


@pytest.mark.parametrize("shape,periodic", [
    ((128, 11, 9), (True, False, False)),    # 64 entries per row: every lane
    ((130, 20, 6), (True, True, True)),      # 65: two wavefronts, one lane in the second
    ((132, 10, 8), (True, True, True)),      # 66: two entries per lane, 33 lanes
    ((256, 21, 6), (False, False, True)),    # 128: two per lane, every lane
    ((260, 10, 12), (False, True, True)),     # 130: two per lane, two wavefronts
    ((264, 31, 4), (True, False, True)),     # 132: four per lane, 33 lanes
    ((512, 14, 6), (True, True, False)),     # 256: four per lane, every lane
    ((520, 13, 5), (False, False, False)),   # 260: four per lane, two wavefronts
    ((646, 6, 4), (True, True, True)),       # 323: one per lane, too many wavefronts
    ((1030, 6, 4), (True, True, True)),      # 515: as above
    ((1288, 5, 3), (False, False, False)),   # 644: four per lane, three wavefronts
    ((64, 130, 200), (True, True, True)),    # ranges that meet two row blocks
    ((66, 67, 300), (False, False, False)),
    ((2, 2, 2), (True, True, True)),
    ((4, 1, 1), (False, False, False)),
])
@pytest.mark.parametrize("precision", [0, 1])
def test_tile_pass_equals_in_place(lb, monkeypatch, shape, periodic, precision):
    case = _case(shape, periodic, 5)
    for iters, rf, every, zeta, solids in ((1, 0.0, 1, True, True), (4, 0.0, 1, False, True),
                                           (7, 0.0, 1, True, True), (6, 1e-9, 3, True, True),
                                           (9, 0.3, 1, False, True), (5, 0.0, 1, False, False)):
        a = _solve(lb, monkeypatch, "1", case, shape, periodic, precision, iters, rf, every, zeta,
                   solids)
        b = _solve(lb, monkeypatch, "0", case, shape, periodic, precision, iters, rf, every, zeta,
                   solids)
        assert a[0] == b[0], (iters, a[0], b[0])
        assert a[2][0] == 1 and b[2][0] == 0
        assert (a[1] == b[1]).all(), (iters, rf, zeta, solids, np.abs(a[1] - b[1]).max())


@pytest.mark.parametrize("periods", [1, 2, 3])
def test_tile_pass_stops_where_it_should(lb, monkeypatch, periods):
    """A residual stop in the middle of a solve: the buffers have been
    swapped an odd or even number of times; the next solve goes on from it."""
    shape, periodic = (96, 22, 18), (True, True, True)
    case = _case(shape, periodic, 8)
    out = {}
    for fused in ("1", "0"):
        monkeypatch.setenv("LBMEP_SOR_FUSED", fused)
        psi, fl, X, R, zv = case
        g = lb.Lattice(shape, periodic, precision=lb.FP32DEV)
        g.set_flags(fl)
        g.set_particles(X, R, np.zeros((len(R), 3)))
        g.set_potential_force(psi, KEPS, (0.0, 0.0, 0.0), zv)
        g.set_potential_solver(0.3, 1.7, 90, 0.05, periods)
        res = [g.solve_potential() for _ in range(3)]
        out[fused] = (res, g.potential())
        g.close()
    assert out["1"][0] == out["0"][0]
    assert (out["1"][1] == out["0"][1]).all()
