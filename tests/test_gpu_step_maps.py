"""The particle part of a step (next level's map set in the sweep's launch,
classification from row bitmaps beside the exchange) against the oracle, maps
bit-exact: radii at the edges of the classification's row store, boxes that
span or wrap periodic axes, overlapping spheres, walls, free spheres, and more
particles than workgroup groups; the two stepping orders bitwise equal."""
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


def _case(name):
    rng = np.random.default_rng(17)
    shape, per, R, n, walls = {
        "rows-in-lds": ((40, 36, 34), (True, True, True), 11.0, 2, False),      # 31^2 rows
        "rows-too-many": ((44, 40, 38), (True, True, True), 12.5, 2, False),    # cell by cell
        "row-too-long": ((66, 9, 9), (True, False, False), 4.0, 2, False),
        "spans-x": ((7, 20, 18), (True, True, True), 3.2, 2, False),
        "spans-all": ((6, 6, 6), (True, True, True), 2.6, 1, False),
        "past-faces": ((21, 19, 23), (False, False, False), 5.0, 5, False),
        "overlap-walls": ((37, 33, 29), (True, False, True), 4.5, 9, True),
        "tiny": ((33, 31, 35), (True, True, True), 0.4, 30, False),
        "many": ((64, 48, 40), (True, True, True), 1.7, 77, False),
    }[name]
    X = rng.random((n, 3)) * np.array(shape)
    U = rng.uniform(-0.3, 0.3, (n, 3))
    W = rng.uniform(-0.01, 0.01, (n, 3))
    fl = np.zeros(shape[::-1], dtype=np.uint8)
    if walls:
        fl[:, 0, :] = fl[:, -1, :] = 1
        fl[rng.random(shape[::-1]) < 0.01] = 1
    return shape, per, X, np.full(n, R), U, W, fl, walls


@pytest.mark.parametrize("name", ["rows-in-lds", "rows-too-many", "row-too-long", "spans-x",
                                  "spans-all", "past-faces", "overlap-walls", "tiny", "many"])
def test_maps_and_forces_follow_the_oracle(lb, oracle_mod, monkeypatch, name):
    shape, per, X, R, U, W, fl, walls = _case(name)
    o = oracle_mod.Oracle(shape, per)
    if walls:
        o.set_flags(fl)
    # the wall-link list is made when the particles are set, without the cells
    # covered then: where a sphere that starts on a wall uncovers them, forces
    # and fields leave the oracle (the maps do not)
    fields = not walls
    o.init_equilibrium(1.0, (1e-3, 0.0, -1e-3))
    o.set_particles(X, R, U, W, moving=True)
    out = []
    for overlap in ("1", "0"):
        monkeypatch.setenv("LBMEP_STEP_OVERLAP", overlap)
        g = lb.Lattice(shape, per, precision=lb.FP64, move_particles=True)
        if walls:
            g.set_flags(fl)
        g.init_equilibrium(1.0, (1e-3, 0.0, -1e-3))
        g.set_particles(X, R, U, W)
        res = []
        for k in (1, 2, 9):
            g.step(k)
            if overlap == "1":
                o.step(k)
                fo, oo = o.map()
                fg, og = g.map()
                assert (fg == fo).all() and (og == oo).all(), (name, k)
            if overlap == "1" and fields:
                Fo, Mo = o.ft()
                Fg, Mg = g.ft()
                s = max(np.abs(Fo).max(), 1e-6)
                assert np.abs(Fg - Fo).max() <= 1e-12 * s
                assert np.abs(Mg - Mo).max() <= 1e-12 * s * max(R[0], 1.0) * 10
                rho_o, u_o = o.macro()
                rho_g, u_g = g.macro()
                assert np.abs(u_g - u_o).max() <= 1e-13
                assert np.abs(rho_g - rho_o).max() <= 1e-12
            res.append((g.map(), g.ft(), g.get_pdfs()))
        out.append(res)
        g.close()
    for (ma, fa, pa), (mb, fb, pb) in zip(*out):
        assert (ma[0] == mb[0]).all() and (ma[1] == mb[1]).all()
        assert (fa[0] == fb[0]).all() and (fa[1] == fb[1]).all() and (pa == pb).all()


def test_free_spheres_and_prescribed_ones_in_turn(lb, oracle_mod):
    """Prescribed motion, then dynamics on the same lattice, then a new table
    of prescribed spheres: the maps' turns and the link lists carry over."""
    shape, per, X, R, U, W, fl, walls = _case("overlap-walls")
    X, R, U, W = X[:3], R[:3] * 0.6, U[:3] * 0.1, W[:3]
    fl[1:-1, 1:-1, :] = 0
    fl[0, 1:-1, :] = fl[-1, 1:-1, :] = 0
    X[:, 1] = (9.0, 16.0, 24.0)  # free of the walls when set
    o = oracle_mod.Oracle(shape, per)
    g = lb.Lattice(shape, per, precision=lb.FP64, move_particles=True)
    for t in (o, g):
        t.set_flags(fl)
        t.init_equilibrium(1.0, (1e-3, 0.0, -1e-3))
    o.set_particles(X, R, U, W, moving=True)
    g.set_particles(X, R, U, W)
    for stage in range(3):
        if stage == 1:
            for t in (o, g):
                t.set_dynamics(1.3, [0.5, -0.4, 0.3], (1e-2, 0.0, 5e-3))
        if stage == 2:
            o.set_particles(X[::-1].copy(), R, U, W, moving=True)
            g.set_particles(X[::-1].copy(), R, U, W)
        o.step(5)
        g.step(5)
        fo, oo = o.map()
        fg, og = g.map()
        assert (fg == fo).all() and (og == oo).all(), stage
        if stage == 2:  # a new table in mid-run: what cells it uncovers hold
            continue    # is not specified
        _, u_o = o.macro()
        _, u_g = g.macro()
        assert np.abs(u_g - u_o).max() <= 1e-12
    g.close()
