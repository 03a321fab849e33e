"""Residual rows between solves: a capped graph-replayed solve whose last
two-sweep pass ran past the budget leaves nothing behind that a later solve
could read."""
import numpy as np
import pytest

from tests.harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("budget", [3, 4])
@pytest.mark.parametrize("fused", [0, 1])
def test_capped_solves_leave_no_rows(budget, fused):
    case = Case(70, 37, 9, Bz=0.1, driven=True, J=0.02, tol=1e-8)
    out = []
    for f in (0, fused):
        s = case.solver()
        s.set_tiling(rows=2, fused=f)
        g = s.step_graph(2, budget, stats=True)
        st = s.step(3)
        out.append((s.get_psi().cpu().numpy(), g["capped_steps"], st["sweeps_sum"]))
        s.close()
    assert out[0][1] == 2 and out[0][1:] == out[1][1:]
    assert np.array_equal(out[0][0], out[1][0])
