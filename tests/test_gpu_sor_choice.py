"""Both sides of the numbers of rows up to which a solve takes the tile pass:
the form changes there and its results do not."""
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


@pytest.mark.parametrize("prec,nx,ny,nz,tile", [
    ("FP32DEV", 6, 500, 250, True), ("FP32DEV", 6, 502, 250, False),          # one entry per lane
    ("FP32DEV", 130, 250, 200, True), ("FP32DEV", 130, 250, 202, False),      # two wavefronts
    ("FP32DEV", 260, 230, 200, True), ("FP32DEV", 260, 230, 202, False),
    ("FP32DEV", 386, 100, 200, True), ("FP32DEV", 386, 100, 202, False),      # four
    ("FP32DEV", 256, 502, 250, True),                                         # any number
    ("FP64", 4, 500, 400, True), ("FP64", 4, 500, 402, False),
    ("FP64", 130, 200, 380, True), ("FP64", 130, 200, 382, False),
    ("FP64", 516, 100, 200, True), ("FP64", 516, 100, 202, False),
    ("FP64", 640, 140, 200, True), ("FP64", 640, 140, 202, False)])
def test_form_and_bits(lb, monkeypatch, prec, nx, ny, nz, tile):
    import torch
    dtype = torch.float64 if prec == "FP64" else torch.float32
    shape = (nx, ny, nz)
    gen = torch.Generator().manual_seed(3)
    psi = torch.rand(nx * ny * nz, generator=gen, dtype=torch.float64).to("cuda", dtype)
    X = np.array([[0.4 * nx, 0.3 * ny, 0.6 * nz], [0.9 * nx, 0.8 * ny, 0.1 * nz]])
    out = []
    for fused in ("1", "0"):
        monkeypatch.setenv("LBMEP_SOR_FUSED", fused)
        L = lb.Lattice(shape, (True, False, True), precision=getattr(lb, prec))
        L.set_particles(X, np.full(2, min(0.4 * nx, 5.0)), np.zeros((2, 3)))
        L.set_potential_force(psi, 1e-3, (0.0, 0.0, 0.0), [0.2, -0.1])
        L.set_potential_solver(0.05, 1.6, 7, 0.0, 1)
        if fused == "1":
            form, rows, planes, _ = L.solver_shape()
            assert form == 1 and (planes == nz) == tile  # the march takes 16 planes at a time
        L.solve_potential()
        got = torch.empty(nx * ny * nz, dtype=torch.float64, device="cuda")
        L.potential(got)
        out.append(got)
        L.close()
    assert torch.equal(out[0], out[1])
