"""Smoothing blocks of the multigrid at the edges of their range: ragged
blocks, axes shorter than a block's halo, odd periodic axes, levels of one
plane, against the exact solution."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1409_8340_amd import inputs, tdgl
from tests.harness import bc_codes, rel_maxerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,open_", [
    ((33, 41, 7), (False, True, True)),      # one node and one plane past a block
    ((64, 72, 1), (False, True, True)),      # one plane
    ((64, 80, 2), (False, True, True)),      # two planes
    ((31, 60, 13), (False, True, True)),     # odd periodic axis shorter than a block
    ((100, 3, 16), (False, True, True)),     # three rows
    ((40, 40, 8), (False, False, False)),    # periodic in all axes
    ((2, 64, 40), (False, True, True)),      # a periodic axis of two nodes
])
def test_smoothing_blocks_vs_exact(shape, open_):
    # FP32 storage of f and mu (6e-8 each, amplified by the spread of the
    # modes, below 100) and the residual stop 1e-7
    import torch
    nx, ny, nz = shape
    grid = O.Grid(nx, ny, nz, 0.5, 0.5, 0.5, open_, 1.0)
    f = inputs.random_real(grid.shape, 41, -1.0, 1.0).astype(np.float64)
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
