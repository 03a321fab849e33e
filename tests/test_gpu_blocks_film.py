"""Block solves of films (four iterates a launch) against single sweeps, bit
for bit: the same film alone, and beside a large idle box that keeps the
context on single sweeps.  The launch counts show which of the two ran."""
import numpy as np
import pytest

from paper_1409_8340_amd import inputs, tdgl
from tests.harness import Case

pytestmark = pytest.mark.gpu


def _pair(case):
    a = case.solver()
    box = tdgl.make_params(1024, 513, 2, bc=(1, 1, 1), max_iter=case.params.max_iter, tol=1e6)
    b = tdgl.Solver([case.params, box])
    case.load_into(b, 0)
    return a, b


def _step(s):
    s.profile_start(["sweep"])
    sweeps = s.step(1)["sweeps_max"]
    return sweeps, s.profile_stop()["sweep"]["launches"]


def _same(a, b, driven, what):
    assert np.array_equal(a.get_psi().cpu().numpy(), b.get_psi(0).cpu().numpy()), what
    if driven:
        assert np.array_equal(a.get_mu().cpu().numpy(), b.get_mu(0).cpu().numpy()), what
        assert a.get_scalars() == b.get_scalars(0), what


@pytest.mark.parametrize("shape,open_,driven,extra", [
    ((96, 50, 1), (False, False, True), True, {}),      # ragged
    ((33, 17, 1), (True, True, True), False, {}),       # one node past a block
    ((64, 48, 1), (True, False, True), False, {}),
    ((3, 2, 1), (False, False, True), True, {}),        # axes shorter than the halo wrap
    ((1, 6, 1), (True, True, True), False, {}),
    ((48, 40, 1), (False, False, True), True, {"noise_T": 0.02, "noise_seed": 5}),
    ((40, 30, 1), (True, False, True), False, {"yz": True}),
    ((40, 30, 1), (False, False, True), True, {"yz": True, "noise_T": 0.02, "noise_seed": 6}),
])
def test_film_blocks_bit_identical_to_single_sweeps(shape, open_, driven, extra):
    nx, ny, nz = shape
    kw = dict(extra)
    yz = kw.pop("yz", False)
    eps = inputs.random_real((nz, ny, nx), 5, 0.4, 1.0)
    kw.update(open_=open_, Bz=0.0 if yz else 0.1, eps=eps, psi_seed=9, driven=driven, J=0.02 if driven else 0.0)
    def start(case):
        a, b = _pair(case)
        if yz:
            for s in (a, b):
                s.set_field_yz(0.1, 0.2, inst=0, quantize=True)
        return a, b
    for tol in (1e-4, 1e-7, 1e-9, 1e-12):
        a, b = start(Case(nx, ny, nz, tol=tol, **kw))
        for rep in range(3):
            (sa, la), (sb, lb) = _step(a), _step(b)
            assert sa == sb
            # single sweeps: a launch per iterate but the first, or more
            # (launches in flight); blocks: a launch per four
            assert lb >= sb - 1
            if sa >= 9:
                assert la < sa - 1
            _same(a, b, driven, (tol, rep))
        a.step_graph(2, 40)
        b.step_graph(2, 40)
        _same(a, b, driven, (tol, "graph"))
        a.close()
        b.close()
    for cap in range(1, 7):
        a, b = start(Case(nx, ny, nz, tol=1e-30, max_iter=cap, **kw))
        a.step(2)
        b.step(2)
        _same(a, b, driven, cap)
        a.close()
        b.close()
