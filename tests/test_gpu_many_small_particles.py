"""Both sides of the number of particles from which a step's exchange takes
smaller workgroups and the classification a launch of its own: against the
oracle, in both stepping orders and the tight form, with dynamics, and
served."""
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


def _case(n, R, walls):
    rng = np.random.default_rng(n)
    shape = (46, 42, 38)
    X = rng.random((n, 3)) * np.array(shape)
    U = rng.uniform(-0.3, 0.3, (n, 3))
    W = rng.uniform(-0.01, 0.01, (n, 3))
    fl = np.zeros(shape[::-1], dtype=np.uint8)
    if walls:
        fl[:, 0, :] = fl[:, -1, :] = 1
    return shape, (True, not walls, True), X, np.full(n, R), U, W, fl


@pytest.mark.parametrize("n", [511, 512, 1300])
@pytest.mark.parametrize("R,walls", [(0.7, True), (1.6, False), (4.0, True), (4.2, False)])
def test_steps_follow_the_oracle(lb, oracle_mod, monkeypatch, n, R, walls):
    """Overlapping spheres crossing the periodic faces: maps bit-exact, forces
    to 1e-12 of the largest (their order of sums is another)."""
    shape, per, X, Rs, U, W, fl = _case(n, R, walls)
    o = oracle_mod.Oracle(shape, per)
    o.set_flags(fl)
    o.init_equilibrium(1.0, (1e-3, 0.0, -1e-3))
    o.set_particles(X, Rs, U, W, moving=True)
    out = []
    for overlap, tight in (("1", "0"), ("0", "0"), ("1", "1")):
        monkeypatch.setenv("LBMEP_STEP_OVERLAP", overlap)
        monkeypatch.setenv("LBMEP_STEP_TIGHT", tight)
        g = lb.Lattice(shape, per, precision=lb.FP64, move_particles=True)
        g.set_flags(fl)
        g.init_equilibrium(1.0, (1e-3, 0.0, -1e-3))
        g.set_particles(X, Rs, U, W)
        res = []
        for k in (1, 1, 6):
            g.step(k)
            if not out:
                o.step(k)
                fo, oo = o.map()
                fg, og = g.map()
                assert (fg == fo).all() and (og == oo).all()
                Fo, Mo = o.ft()
                Fg, Mg = g.ft()
                s = max(np.abs(Fo).max(), 1e-6)
                assert np.abs(Fg - Fo).max() <= 1e-12 * s
                assert np.abs(Mg - Mo).max() <= 1e-11 * s * max(R, 1.0)
                assert np.abs(g.macro()[1] - o.macro()[1]).max() <= 1e-13
            res.append((*g.map(), *g.ft(), g.get_pdfs()))
        out.append(res)
        g.close()
    for a, b, c in zip(*out):
        for x, y, z in zip(a, b, c):
            assert (x == y).all() and (x == z).all()


@pytest.mark.parametrize("n", [511, 512])
def test_free_spheres(lb, oracle_mod, n):
    """Heavy ones (their velocity changes by F / m of 1e-3): positions within
    1e-12."""
    shape, per, X, R, U, W, fl = _case(n, 1.6, False)
    o = oracle_mod.Oracle(shape, per)
    g = lb.Lattice(shape, per, precision=lb.FP64, move_particles=True)
    for t in (o, g):
        t.init_equilibrium(1.0, (1e-3, 0.0, -1e-3))
    o.set_particles(X, R, 0.5 * U, W, moving=True)
    g.set_particles(X, R, 0.5 * U, W)
    for t in (o, g):
        t.set_dynamics(500.0, np.full(n, 1.0), (1e-2, 0.0, 5e-3))
        t.step(6)
    assert (g.map()[0] == o.map()[0]).all() and (g.map()[1] == o.map()[1]).all()
    for a, b in zip(g.particles(), o.particles()):
        assert np.abs(a - b).max() <= 1e-12 * max(1.0, np.abs(b).max())
    g.close()


def test_served_in_one_mix(lb):
    """Few and many particles, moving and fixed, two radii: bitwise as alone."""
    srv = lb.Server(2 << 30, max_slots=8, chunk_steps=4)
    want = {}
    for k, (n, R, moving) in enumerate([(511, 1.6, True), (512, 1.6, True), (1100, 5.0, True),
                                        (1200, 0.7, False), (3, 4.0, True)]):
        shape, per, X, Rs, U, W, fl = _case(n, R, k % 2 == 0)
        kw = dict(periodic=per, X=X, R=Rs, U=0.1 * U, W=W, steps=6 + 3 * k, flags=fl,
                  precision=lb.FP32DEV, moving=moving, keep_fields=True)
        want[srv.submit(shape, **kw)] = (shape, kw)
    srv.wait_all(list(want), sleep=0.0)
    for i, (shape, kw) in want.items():
        L = lb.Lattice(shape, kw["periodic"], precision=lb.FP32DEV, move_particles=kw["moving"])
        L.set_flags(kw["flags"])
        L.set_particles(kw["X"], kw["R"], kw["U"], kw["W"])
        L.step(kw["steps"])
        rho, u = L.macro()
        F, M = L.ft()
        L.close()
        got, res = srv.fields(i), srv.result(i)
        assert (got[0] == rho).all() and (got[1] == u).all()
        assert (res[0] == F).all() and (res[1] == M).all()
    srv.close()
