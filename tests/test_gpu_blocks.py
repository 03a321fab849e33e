"""Block solves (several Jacobi iterations per launch on small grids) against
single sweeps, bit for bit: the same instance alone takes blocks, and beside a
large idle instance in one context takes single sweeps."""
import numpy as np
import pytest

from paper_1409_8340_amd import inputs, tdgl
from tests.harness import Case

pytestmark = pytest.mark.gpu

CASES = [
    # shape, open, Bx, Bz, driven, extra
    # small blocks 16 x 8 x 2: ragged, every face kind, one block and less
    ((70, 37, 9), (False, False, True), 0.0, 0.1, True, {}),
    ((40, 24, 12), (True, True, True), 0.2, 0.3, False, {}),
    ((17, 9, 3), (False, False, False), 0.1, 0.1, False, {}),
    ((16, 8, 2), (False, False, True), 0.0, 0.2, True, {}),
    ((5, 3, 4), (False, False, False), 0.0, 0.3, False, {}),    # axes shorter than the halo wrap
    ((2, 2, 2), (False, False, True), 0.0, 0.4, True, {}),
    ((1, 6, 1), (True, True, True), 0.0, 0.2, False, {}),       # one-node open axes
    ((6, 1, 3), (True, True, False), 0.1, 0.0, False, {}),
    ((33, 18, 7), (False, True, True), 0.15, 0.1, True, {}),
    ((50, 20, 6), (False, False, True), 0.0, 0.1, True, {"noise_T": 0.02, "noise_seed": 9}),
    # blocks 32 x 8 x 4: above 128 K nodes
    ((97, 45, 33), (False, False, True), 0.1, 0.1, False, {}),
    ((64, 48, 45), (True, False, False), 0.0, 0.1, False, {}),
    # films: blocks 32 x 16, four iterates a launch
    ((96, 50, 1), (False, False, True), 0.0, 0.1, True, {}),
    ((33, 17, 1), (True, True, True), 0.0, 0.1, False, {}),
    ((3, 2, 1), (False, False, True), 0.0, 0.1, False, {}),
    ((48, 40, 1), (False, False, True), 0.0, 0.1, True, {"noise_T": 0.02, "noise_seed": 5}),
]


def _pair(case):
    """(alone: blocks, beside 1.05 M idle nodes: single sweeps)"""
    a = case.solver()
    filler = tdgl.make_params(1024, 1025, 1, bc=(1, 1, 1), max_iter=case.params.max_iter, tol=1e6)
    b = tdgl.Solver([case.params, filler])
    case.load_into(b, 0)
    return a, b


def _same(a, b, driven, what):
    assert np.array_equal(a.get_psi().cpu().numpy(), b.get_psi(0).cpu().numpy()), what
    if driven:
        assert np.array_equal(a.get_mu().cpu().numpy(), b.get_mu(0).cpu().numpy()), what
        assert a.get_scalars() == b.get_scalars(0), what


@pytest.mark.parametrize("shape,open_,Bx,Bz,driven,extra", CASES)
def test_blocks_bit_identical_to_single_sweeps(shape, open_, Bx, Bz, driven, extra):
    nx, ny, nz = shape
    eps = inputs.random_real((nz, ny, nx), 5, 0.4, 1.0)
    kw = dict(open_=open_, Bx=Bx, Bz=Bz, eps=eps, psi_seed=9, driven=driven, J=0.02 if driven else 0.0, **extra)
    # sweep counts of every residue: eager steps follow the recent counts
    for tol in (1e-4, 1e-6, 1e-7, 1e-9, 1e-10):
        a, b = _pair(Case(nx, ny, nz, tol=tol, **kw))
        sweeps = 0
        for rep in range(3):
            sweeps += a.step(1)["sweeps_sum"]
            b.step(1)
            _same(a, b, driven, (tol, rep))
        a.step_graph(2, 30)
        b.step_graph(2, 30)
        _same(a, b, driven, (tol, "graph"))
        a.close()
        b.close()
    # caps inside a launch
    for cap in range(1, 7):
        c = Case(nx, ny, nz, tol=1e-30, max_iter=cap, **kw)
        a, b = _pair(c)
        sa = a.step(2)
        b.step(2)
        assert sa["capped_steps"] == 2 and sa["sweeps_sum"] == 2 * cap and sa["sweep_passes"] == 2 * (cap - 1)
        _same(a, b, driven, cap)
        a.step_graph(1, 1)
        b.step_graph(1, 1)
        _same(a, b, driven, (cap, "graph"))
        a.close()
        b.close()


@pytest.mark.parametrize("shape,open_", [((48, 24, 10), (False, False, True)), ((40, 30, 1), (True, False, True))])
def test_blocks_yz_field(shape, open_):
    nx, ny, nz = shape
    c = Case(nx, ny, nz, open_=open_, tol=1e-9, psi_seed=3)
    a, b = _pair(c)
    for s in (a, b):
        s.set_field_yz(0.1, 0.2, inst=0, quantize=True)
    for rep in range(3):
        a.step(1)
        b.step(1)
        _same(a, b, False, rep)
    a.close()
    b.close()


def test_blocks_in_an_uneven_batch():
    cases = [Case(16, 12, 4, Bz=0.2, tol=1e-6, psi_seed=1), Case(40, 33, 5, Bz=0.1, tol=1e-10, psi_seed=2),
             Case(20, 16, 9, Bz=0.3, tol=1e-8, max_iter=5, psi_seed=4)]
    s = tdgl.Solver([c.params for c in cases])
    for i, c in enumerate(cases):
        c.load_into(s, i)
    s.step(2)
    s.step_graph(2, 20)
    for i, c in enumerate(cases):
        a, b = _pair(c)
        b.step(2)
        b.step_graph(2, min(20, c.params.max_iter))
        assert np.array_equal(s.get_psi(i).cpu().numpy(), b.get_psi(0).cpu().numpy()), i
        a.close()
        b.close()
    s.close()
