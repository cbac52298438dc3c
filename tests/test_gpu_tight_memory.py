"""The form of a lattice without the third map, the bitmaps and the second set
of link lists: same results as the usual one, and requests that fit a server's
budget only in it are served."""
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


def _state(g):
    return [g.map()[0], g.map()[1], *g.ft(), *g.macro(), *g.particles(), g.get_pdfs()]


@pytest.mark.parametrize("prec", ["FP64", "FP16DEV"])
@pytest.mark.parametrize("motion", ["fixed", "prescribed", "free", "both in turn"])
def test_tight_lattice_gives_the_same_bits(lb, monkeypatch, tmp_path, motion, prec):
    rng = np.random.default_rng(8)
    shape, per = (34, 31, 28), (True, False, False)
    fl = np.zeros(shape[::-1], dtype=np.uint8)
    fl[:, 0, :] = 1
    fl[rng.random(shape[::-1]) < 0.003] = 1
    n = 7
    X = rng.random((n, 3)) * np.array(shape)
    R = rng.uniform(0.6, 5.0, n)
    U = rng.uniform(-0.01, 0.01, (n, 3)) if prec == "FP16DEV" else rng.uniform(-0.3, 0.3, (n, 3))
    out = []
    for tight in ("0", "1"):
        monkeypatch.setenv("LBMEP_STEP_TIGHT", tight)
        g = lb.Lattice(shape, per, precision=getattr(lb, prec), move_particles=motion != "fixed")
        g.set_flags(fl)
        g.set_free_slip([0, 0, 0, 0, 1, 1])
        g.set_particles(X, R, U, 0.1 * U)
        if motion == "free":
            g.set_dynamics(80.0, np.full(n, 2.0), (1e-3, -2e-3, 1e-3))
        res = []
        for k in (1, 2, 3, 5):
            g.step(k)
            res.append(_state(g))
        if motion == "both in turn":
            g.set_dynamics(80.0, np.full(n, 2.0), (1e-3, -2e-3, 1e-3))
            g.step(4)
            res.append(_state(g))
            g.set_particles(X[::-1].copy(), 1.2 * R, U)
            g.step(3)
            res.append(_state(g))
        path = str(tmp_path / f"state{tight}")
        g.save(path)
        g.step(2)
        h = lb.Lattice(shape, per, precision=getattr(lb, prec), move_particles=motion != "fixed")
        h.load(path)
        h.step(2)
        for a, b in zip(_state(g), _state(h)):
            assert (a == b).all()
        res.append(_state(h))
        out.append(res)
        g.close()
        h.close()
    for ra, rb in zip(*out):
        for a, b in zip(ra, rb):
            assert (a == b).all()


@pytest.mark.parametrize("moving", [True, False])
def test_request_that_fits_only_without_them_is_served(lb, moving):
    """Beside others that need not do without, and alone."""
    rng = np.random.default_rng(3)
    shape = (72, 70, 66)
    N = shape[0] * shape[1] * shape[2]
    X = rng.random((12, 3)) * np.array(shape)
    kw = dict(X=X, R=np.full(12, 3.5), U=rng.uniform(-0.02, 0.02, (12, 3)), steps=23,
              rho_e=(rng.random(N) * 1e-4).astype(np.float32), E=(1e-3, 0.0, 2e-3),
              precision=lb.FP32DEV, moving=moving, keep_fields=True)
    less = 4 * N if moving else N // 4  # the third map; the bitmaps
    srv = lb.Server(lb.Server.request_footprint(shape, **kw) - less, max_slots=4, chunk_steps=5)
    small = (20, 18, 16)
    skw = dict(X=np.array([[9.0, 8.5, 7.0]]), R=[3.0], U=[[0.01, 0.0, 0.0]], steps=31,
               precision=lb.FP32DEV, moving=True, keep_fields=True)
    ids = [srv.submit(small, **skw), srv.submit(shape, **kw), srv.submit(small, **skw)]
    srv.wait_all(ids, sleep=0.0)
    for i, (s, q) in zip(ids, [(small, skw), (shape, kw), (small, skw)]):
        L = lb.Lattice(s, precision=lb.FP32DEV, move_particles=q["moving"])
        if "rho_e" in q:
            L.set_charge_force(q["rho_e"], q["E"])
        L.set_particles(q["X"], q["R"], q["U"])
        L.step(q["steps"])
        rho, u = L.macro()
        F, M = L.ft()
        inv = L.invariants()
        L.close()
        got = srv.fields(i)
        assert (got[0] == rho).all() and (got[1] == u).all()
        res = srv.result(i)
        assert (res[0] == F).all() and (res[1] == M).all() and (res[2] == inv).all()
    srv.close()
