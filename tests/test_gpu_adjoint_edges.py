"""The reverse step's own neighbour sums at the edges of their range: axes of
one and two nodes, ragged ends of the flat passes, and fields on open and
periodic faces, against the oracle's adjoint."""
import numpy as np
import pytest

from oracle import adjoint as A
from tests.harness import Case
from tests.test_gpu_adjoint import _compare, _eps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,open_,Bx", [
    ((12, 8, 1), (False, False, True), 0.0),    # a film
    ((12, 2, 5), (False, False, True), 0.0),    # both y neighbours the same node
    ((12, 2, 4), (False, True, True), 0.0),     # open y of two nodes: each the other's ghost
    ((10, 7, 2), (False, True, True), 0.1),     # open z of two nodes
    ((2, 6, 3), (False, False, True), 0.1),     # both x neighbours the same node
    ((40, 31, 9), (False, False, True), 0.1),   # a ragged last work-group
])
def test_reverse_step_edges(shape, open_, Bx):
    nx, ny, nz = shape
    case = Case(nx, ny, nz, open_=open_, Bz=0.2, Bx=Bx, J=0.06, driven=True, tol=1e-12, max_iter=250, mu_tol=1e-7,
                mu_max_cycles=60, eps=_eps((nz, ny, nx), 31), psi_seed=32)
    s = case.solver()
    v, g = s.voltage_grad(4, 1, ckpt_every=3)
    g = g.cpu().numpy()
    s.close()
    V_o, g_o = A.voltage_grad(case.grid, case.oracle_params("exact"), case.eps.astype(np.float64),
                              case.oracle_state(), 4, 1)
    rel, cos = _compare(g, g_o)
    print(f"[adjoint {shape} {open_}] Vbar gpu {v:.8e} oracle {V_o:.8e}; grad rel L2 {rel:.3e} cos {cos:.6f}")
    assert np.isfinite(g).all()
    # FP32 forward and iterative solves against the exact FP64 step: the
    # bounds of the larger boxes
    assert abs(v - V_o) <= 1e-3 * abs(case.J)
    assert rel <= 1e-2 and cos >= 0.9999
