"""More particle workgroups in a step than the 32-bit thread count of a grid's
x extent holds (three of 512 threads per moving sphere): every sphere still
takes part."""
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


def _lattice(lb, m, overlap, monkeypatch):
    """m^3 spheres of one cell each, three cells apart."""
    monkeypatch.setenv("LBMEP_STEP_OVERLAP", overlap)
    L = lb.Lattice((3 * m,) * 3, precision=lb.FP16DEV, move_particles=True)
    i = 1.5 + 3.0 * np.arange(m)
    z, y, x = np.meshgrid(i, i, i, indexing="ij")
    X = np.stack([x, y, z], axis=-1).reshape(-1, 3)
    n = len(X)
    L.set_particles(X, np.full(n, 0.6), np.tile([[2e-3, 0.0, -1e-3]], (n, 1)))
    L.step(3)
    return L


@pytest.mark.parametrize("overlap", ["1", "0"])
def test_every_sphere_of_a_periodic_pattern_does_the_same(lb, monkeypatch, overlap):
    """141^3 spheres (8.4 million workgroups) against 2^3 of the same pattern:
    the same values in every cell and on every link, so forces equal up to the
    rounding of the positions (1e-12), and exactly as many obstacle cells."""
    m = 141
    assert 3 * m ** 3 * 512 > 2 ** 32
    small, large = _lattice(lb, 2, overlap, monkeypatch), _lattice(lb, m, overlap, monkeypatch)
    F0, _ = small.ft()
    F, _ = large.ft()
    assert np.abs(F0).max() > 0.0
    assert np.abs(F - F0[0]).max() <= 1e-12 * np.abs(F0).max()
    fl, ow = large.map()
    assert (ow.reshape(-1)[ow.reshape(-1) >= 0] == np.arange(m ** 3)).all()
    f0, _ = small.map()
    assert (np.tile(f0[:3, :3, :3], (m, m, m)) == fl).all()
    small.close()
    large.close()
