"""Fields of served requests that are held while more finish than the server's
pinned blocks have room for, and blocks used again by results of other sizes."""
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


def _alone(lb, shape, X, R, U, steps, rho_e):
    L = lb.Lattice(shape, precision=lb.FP32DEV, move_particles=True)
    L.set_charge_force(rho_e, (1e-3, 0.0, 2e-3))
    L.set_particles(X, R, U)
    L.step(steps)
    out = L.macro()
    L.close()
    return out


@pytest.mark.parametrize("budget_mb", [40, 400])
def test_held_results_keep_their_fields(lb, budget_mb):
    """Bitwise what a lattice of its own gives (budget 40 MB: one request of
    48^3 at a time, room for about ten of its 3.5 MB results)."""
    srv = lb.Server(budget_mb << 20, max_slots=4)
    rng = np.random.default_rng(1)
    held = {}
    for wave, edge in enumerate((48, 48, 24, 40)):
        ids = []
        for r in range(14):
            shape = (edge, edge, edge - 8 * (r % 2))
            N = shape[0] * shape[1] * shape[2]
            X = np.array([[0.5 * s for s in shape]]) + rng.random((1, 3))
            kw = dict(X=X, R=np.array([3.0 + 0.1 * r]), U=np.full((1, 3), 1e-3))
            rho_e = (rng.random(N) * 1e-4).astype(np.float32)
            i = srv.submit(shape, steps=2 + r % 3, rho_e=rho_e, E=(1e-3, 0.0, 2e-3),
                           precision=lb.FP32DEV, moving=True, keep_fields=True, **kw)
            held[i] = (shape, kw["X"], kw["R"], kw["U"], 2 + r % 3, rho_e)
            ids.append(i)
        srv.wait_all(ids, sleep=0.0)
        if wave == 1:
            continue  # held beside the next wave's
        for i in list(held):
            rho, u = srv.fields(i)
            ref = _alone(lb, *held[i])
            assert (rho == ref[0]).all() and (u == ref[1]).all(), (wave, i)
            srv.release(i)
            del held[i]
    srv.close()


@pytest.mark.parametrize("prec", ["FP64", "FP32DEV"])
def test_batch_larger_than_the_infinity_cache(lb, prec):
    """Batches whose populations start above the cache's size and fall below
    it as requests finish (FP64 64^3: 80 MB each): the sweep's streaming hints
    change on the way, the results do not."""
    precision = getattr(lb, prec)
    edges = (64, 64, 60, 64, 62) if prec == "FP64" else (80, 84, 80, 82, 80)
    srv = lb.Server(2 << 30, max_slots=8, chunk_steps=2)
    rng = np.random.default_rng(4)
    want = {}
    for r, e in enumerate(edges):
        shape, steps = (e, e - 6, e + 2), 3 + 2 * r
        X = rng.random((3, 3)) * np.array(shape)
        U = rng.uniform(-0.01, 0.01, (3, 3))
        R = np.array([3.0, 4.0, 3.5])
        i = srv.submit(shape, X=X, R=R, U=U, steps=steps, precision=precision, moving=True,
                       keep_fields=True)
        want[i] = (shape, X, R, U, steps)
    srv.wait_all(list(want), sleep=0.0)
    for i, (shape, X, R, U, steps) in want.items():
        L = lb.Lattice(shape, precision=precision, move_particles=True)
        L.set_particles(X, R, U)
        L.step(steps)
        rho, u = L.macro()
        got = srv.fields(i)
        assert (got[0] == rho).all() and (got[1] == u).all()
        F, M = L.ft()
        res = srv.result(i)
        assert (res[0] == F).all() and (res[1] == M).all()
        L.close()
        srv.release(i)
    srv.close()
