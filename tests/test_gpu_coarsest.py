"""The multigrid's coarsest level, where that level is the whole grid:
tdgl_poisson_solve against the oracle's exact solution."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1409_8340_amd import inputs, tdgl
from tests.harness import bc_codes, rel_maxerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,open_,g,hy", [
    ((64, 4, 2), (False, True, True), 1.0, 0.5),
    ((63, 4, 2), (False, True, True), 1.0, 0.5),     # odd periodic axis
    ((65, 3, 2), (False, True, True), 1.0, 0.5),
    ((15, 13, 11), (False, False, False), 1.0, 0.5),  # more nodes than threads: no axis coarsens
    ((8, 8, 8), (False, False, False), 2.0, 0.4),    # all periodic, anisotropic
    ((2, 64, 4), (False, True, True), 1.0, 0.3),     # two nodes on a periodic axis
    ((7, 1, 1), (False, True, True), 1.0, 0.5),      # one-node open axes
    ((1, 5, 9), (False, True, True), 0.5, 0.5),      # one-node periodic axis
    ((2, 2, 1), (False, True, True), 1.0, 0.5),
    ((192, 13, 9), (False, True, True), 1.0, 0.5),   # below four finer levels
])
def test_coarsest_level_vs_exact(shape, open_, g, hy):
    # FP32 storage of f and mu (6e-8 each, amplified by the spread of the
    # modes, below 100 here) and the residual stop 1e-7
    import torch
    nx, ny, nz = shape
    grid = O.Grid(nx, ny, nz, 0.5, hy, 0.5, open_, g)
    f = inputs.random_real(grid.shape, 37, -1.0, 1.0).astype(np.float64)
    w = O.node_weights(grid)
    f -= np.sum(w * f) / np.sum(w)
    ref = O.poisson_exact(grid, f)
    p = tdgl.make_params(nx, ny, nz, hy=hy, bc=bc_codes(open_), g=g, driven=True, mu_tol=1e-7, mu_max_cycles=60,
                         poisson=1)
    s = tdgl.Solver(p)
    mu = s.poisson_solve(torch.from_numpy(f.astype(np.float32)).cuda()).cpu().numpy()
    s.close()
    err = rel_maxerr(mu, ref)
    print(shape, open_, "rel err", err)
    assert err <= 2e-5
