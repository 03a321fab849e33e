"""Single sweeps and the assemble at the edges of their tiles and z runs, bit
for bit against block solves of the same instance: one and two planes on open
and periodic z axes, a column more or less than a tile, rows off the grid."""
import numpy as np
import pytest

from paper_1409_8340_amd import tdgl
from tests.harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 2, 4])
@pytest.mark.parametrize("shape,open_", [
    ((64, 8, 1), (False, False, True)),
    ((65, 9, 1), (False, False, False)),     # one plane, its own z neighbour
    ((63, 17, 1), (True, True, True)),
    ((66, 15, 2), (False, False, True)),
    ((129, 16, 2), (True, False, False)),
    ((72, 7, 3), (False, True, True)),
    ((1, 33, 5), (True, False, True)),
    ((40, 1, 4), (False, True, False)),
])
def test_single_sweeps_at_tile_edges(shape, open_, rows):
    nx, ny, nz = shape
    c = Case(nx, ny, nz, open_=open_, Bx=0.1 if open_[2] else 0.0, Bz=0.2, tol=1e-9, psi_seed=7)
    a = c.solver()
    # a box of 2^20 nodes beside it keeps the context on single sweeps
    b = tdgl.Solver([c.params, tdgl.make_params(256, 256, 17, bc=(1, 1, 1), max_iter=200, tol=1e6)])
    b.set_tiling(rows=rows)
    c.load_into(b, 0)
    for rep in range(2):
        a.step(1)
        b.step(1)
        assert np.array_equal(a.get_psi().cpu().numpy(), b.get_psi(0).cpu().numpy()), rep
    a.close()
    b.close()
