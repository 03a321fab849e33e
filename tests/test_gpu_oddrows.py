"""Spectral Poisson solve with an odd number of rows, whose row pairs run on
across planes: against the exact solution, and beside even ones in a batch."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1409_8340_amd import inputs, tdgl
from tests.harness import bc_codes, rel_maxerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(16, 15, 8), (30, 9, 7), (12, 1, 5), (64, 27, 1), (100, 81, 20), (8, 75, 67),
                                   (20, 125, 140), (1080, 5, 3)])
def test_odd_rows_vs_exact(shape):
    # a direct solve: FP32 storage of f and mu and FP32 transforms of up to
    # 1080 x 125 points (a few 1e-7 of the largest value)
    import torch
    nx, ny, nz = shape
    open_ = (False, False, True)
    grid = O.Grid(nx, ny, nz, 0.5, 0.5, 0.5, open_, 1.0)
    f = inputs.random_real(grid.shape, 43, -1.0, 1.0).astype(np.float64)
    w = O.node_weights(grid)
    f -= np.sum(w * f) / np.sum(w)
    ref = O.poisson_exact(grid, f)
    p = tdgl.make_params(nx, ny, nz, bc=bc_codes(open_), driven=True)
    s = tdgl.Solver(p)
    mu = s.poisson_solve(torch.from_numpy(f.astype(np.float32)).cuda()).cpu().numpy()
    s.close()
    err = rel_maxerr(mu, ref)
    print(shape, "rel err", err)
    assert err <= 5e-6


def test_odd_beside_even_in_a_batch():
    import torch
    shapes = [(30, 15, 6), (32, 16, 8), (24, 27, 5)]
    def start(s, i, n):
        s.set_field(0.0, 0.1, inst=i)
        s.set_current(0.05, inst=i)
        psi = inputs.random_complex((n[2], n[1], n[0]), 5 + n[0], 0.5).astype(np.complex64)
        s.set_psi(torch.from_numpy(psi).cuda(), inst=i)
    b = tdgl.Solver([tdgl.make_params(*n, driven=True, max_iter=60, tol=1e-10) for n in shapes])
    for i, n in enumerate(shapes):
        start(b, i, n)
    b.step(3)
    for i, n in enumerate(shapes):
        a = tdgl.Solver(tdgl.make_params(*n, driven=True, max_iter=60, tol=1e-10))
        start(a, 0, n)
        a.step(3)
        assert np.array_equal(a.get_psi(0).cpu().numpy(), b.get_psi(i).cpu().numpy()), n
        assert np.array_equal(a.get_mu(0).cpu().numpy(), b.get_mu(i).cpu().numpy()), n
        a.close()
    b.close()
