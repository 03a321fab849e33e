"""Eager steps of batches whose instances differ in max_iter: one instance
stops at its cap while another iterates on, wherever the cap falls within a
launch.  The capped instance ends on the bits it has alone."""
import numpy as np
import pytest

from paper_1409_8340_amd import tdgl
from tests.harness import Case

pytestmark = pytest.mark.gpu

BOX = ((24, 18, 6), (20, 12, 5))
FILM = ((40, 33, 1), (32, 20, 1))
TILES = ((128, 64, 4), (70, 37, 5))    # all super-tiles, and boundary tiles


@pytest.mark.parametrize("shapes,fused", [(BOX, 0), (FILM, 0), (TILES, 1), (TILES[::-1], 1)],
                         ids=["blocks", "films", "two_sweep", "two_sweep_boundary"])
@pytest.mark.parametrize("tol", [1e-30, 1e-6, 1e-8, 1e-10])
def test_cap_beside_a_longer_solve(shapes, fused, tol):
    # tol: of the longer solve, whose sweep counts choose where launches start
    for cap in range(1, 10):
        cases = [Case(*shapes[0], Bz=0.2, tol=1e-30, max_iter=cap, psi_seed=1),
                 Case(*shapes[1], Bz=0.3, tol=tol, max_iter=24, psi_seed=2)]
        s = tdgl.Solver([c.params for c in cases])
        alone = [c.solver() for c in cases]
        if fused:
            s.set_tiling(rows=2, fused=1)
        for i, c in enumerate(cases):
            c.load_into(s, i)
        for rep in range(4):
            st = s.step(1)
            own = [a.step(1) for a in alone]
            assert st["sweeps_sum"] == own[0]["sweeps_sum"] + own[1]["sweeps_sum"], (cap, rep)
            assert own[0]["sweeps_sum"] == cap
            for i, a in enumerate(alone):
                assert np.array_equal(a.get_psi().cpu().numpy(), s.get_psi(i).cpu().numpy()), (cap, rep, i)
        for x in (s, *alone):
            x.close()
