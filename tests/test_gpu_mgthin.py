"""Multigrid on long thin boxes, whose level tables are large beside their
values: the tail ends by LDS instead of nodes, or reads its table from memory
where a long axis cannot be halved."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1409_8340_amd import inputs, tdgl
from tests.harness import bc_codes

pytestmark = pytest.mark.gpu

OPEN = (False, True, True)


@pytest.mark.parametrize("shape", [
    (4096, 1, 1),    # the tail starts at 1024 nodes
    (4096, 2, 1),    # at 2048
    (3200, 1, 1),
    (8190, 1, 1),    # coarsest level 4095 x 1 x 1: its table alone exceeds LDS
])
def test_thin_box_residual(shape):
    # right side of short waves (nx / 16 and nx / 12 periods), which the coarse
    # Jacobi sweeps reduce quickly: the stop rule has to be met, so the residual
    # of the returned mu is the stop's 1e-5 and the rounding of mu to FP32,
    # |mu| <= 2.7 (twice the larger wave's 1 / 0.61 + the other's, rounded up
    # from 2.6), 2.7 * 2^-24 * (4 / h^2 + 4 / h^2) = 5.2e-6
    import torch
    nx, ny, nz = shape
    grid = O.Grid(nx, ny, nz, 0.5, 0.5, 0.5, OPEN, 1.0)
    x = np.arange(nx)
    f = np.cos(2 * np.pi * (nx // 16) * x / nx) + np.sin(2 * np.pi * (nx // 12) * x / nx)
    f = np.broadcast_to(f, grid.shape).astype(np.float32)
    p = tdgl.make_params(nx, ny, nz, bc=bc_codes(OPEN), driven=True, mu_tol=1e-5, mu_max_cycles=60, poisson=1)
    s = tdgl.Solver(p)
    mu = s.poisson_solve(torch.from_numpy(f.copy()).cuda()).cpu().numpy().astype(np.float64)
    s.close()
    assert np.max(np.abs(mu)) <= 2.7
    w = O.node_weights(grid)
    f = f - np.sum(w * f) / np.sum(w)
    res = float(np.max(np.abs(f - O.poisson_apply(grid, mu))))
    print(shape, "residual", res)
    assert res <= 1.52e-5
    assert abs(np.sum(w * mu) / np.sum(w)) <= 2.7e-7


def test_thin_boxes_beside_others():
    shapes = [(8190, 1, 1), (34, 31, 33), (4096, 1, 1), (8, 5, 4)]
    def params(n):
        return tdgl.make_params(*n, bc=bc_codes(OPEN), driven=True, mu_tol=1e-5, mu_max_cycles=4, poisson=1,
                                max_iter=60, tol=1e-10)
    def start(s, i, n):
        import torch
        psi = inputs.random_complex((n[2], n[1], n[0]), 11 + n[0], 0.5).astype(np.complex64)
        s.set_field(0.0, 0.1, inst=i)
        s.set_current(0.05, inst=i)
        s.set_psi(torch.from_numpy(psi).cuda(), inst=i)
    b = tdgl.Solver([params(n) for n in shapes])
    for i, n in enumerate(shapes):
        start(b, i, n)
    b.step(2)
    for i, n in enumerate(shapes):
        a = tdgl.Solver(params(n))
        start(a, 0, n)
        a.step(2)
        assert np.array_equal(a.get_psi(0).cpu().numpy(), b.get_psi(i).cpu().numpy()), n
        assert np.array_equal(a.get_mu(0).cpu().numpy(), b.get_mu(i).cpu().numpy()), n
        a.close()
    b.close()
