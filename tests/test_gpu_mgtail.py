"""The multigrid's coarse end in one work-group: tails of one and several
levels against the exact solution, and instances of unlike depth in a batch
against the same instances alone."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1409_8340_amd import inputs, tdgl
from tests.harness import bc_codes, rel_maxerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,open_", [
    ((21, 25, 9), (False, True, True)),      # 4725 nodes above the tail, odd periodic axis
    ((16, 16, 16), (False, True, True)),     # tail right below the finest level
    ((34, 31, 33), (False, True, True)),     # two levels above it
    ((17, 40, 1), (False, True, True)),
])
def test_tail_vs_exact(shape, open_):
    # FP32 storage of f and mu (6e-8 each, amplified by the spread of the
    # modes, below 100) and the residual stop 1e-7
    import torch
    nx, ny, nz = shape
    grid = O.Grid(nx, ny, nz, 0.5, 0.5, 0.5, open_, 1.0)
    f = inputs.random_real(grid.shape, 37, -1.0, 1.0).astype(np.float64)
    w = O.node_weights(grid)
    f -= np.sum(w * f) / np.sum(w)
    ref = O.poisson_exact(grid, f)
    p = tdgl.make_params(nx, ny, nz, bc=bc_codes(open_), driven=True, mu_tol=1e-7, mu_max_cycles=60, poisson=1)
    s = tdgl.Solver(p)
    mu = s.poisson_solve(torch.from_numpy(f.astype(np.float32)).cuda()).cpu().numpy()
    s.close()
    err = rel_maxerr(mu, ref)
    print(shape, "rel err", err)
    assert err <= 2e-5


def test_unlike_depths_in_a_batch():
    shapes = [(34, 31, 33), (8, 5, 4), (64, 40, 12), (16, 16, 16)]
    def params(n):
        return tdgl.make_params(*n, bc=bc_codes((False, True, True)), driven=True, mu_tol=1e-5, mu_max_cycles=20,
                                poisson=1, max_iter=60, tol=1e-10)
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
