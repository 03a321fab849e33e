"""Two forms of the same pass: the fused y and z pass of the spectral solve
against the separate passes that a context takes beside an instance too large
for it, and the residual maximum of blocks and single sweeps with a NaN in
psi."""
import numpy as np
import pytest

from paper_1409_8340_amd import inputs, tdgl
from tests.harness import Case, rel_maxerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(32, 16, 6), (27, 25, 17), (20, 32, 65), (48, 40, 1), (10, 1, 7), (6, 12, 256)])
def test_fused_yz_against_separate_passes(shape):
    # the same FP32 transforms; the z systems in FP64, summed in another order
    # and rounded once: a bin may round the other way, 2^-23 of itself, and
    # the largest bin is no larger than the largest |mu| times what it spreads to
    nx, ny, nz = shape
    mu0 = inputs.random_real((nz, ny, nx), 6, -0.05, 0.05)
    c = Case(nx, ny, nz, Bz=0.1, J=0.05, driven=True, mu0=mu0, K0=0.3, tol=1e-10)
    c.psi0 = inputs.random_complex((nz, ny, nx), 8, 0.5)
    a = c.solver()
    big = tdgl.make_params(8, 640, 32, driven=True, tol=1e6)    # 20480 points per kx plane
    b = tdgl.Solver([c.params, big])
    c.load_into(b, 0)
    for rep in range(2):
        a.step(1)
        b.step(1)
        assert rel_maxerr(b.get_mu(0).cpu().numpy(), a.get_mu().cpu().numpy()) <= 2.0 ** -22, rep
    a.close()
    b.close()


@pytest.mark.parametrize("shape", [(40, 24, 12), (66, 65, 64), (96, 50, 1)])
def test_nan_keeps_the_solve_open(shape):
    # a NaN residual meets no tolerance: every kernel runs into the cap
    import torch
    nx, ny, nz = shape
    psi = inputs.random_complex((nz, ny, nx), 9, 0.5).astype(np.complex64)
    psi[nz // 2, ny // 2, nx // 3] = np.nan
    p = tdgl.make_params(nx, ny, nz, tol=1e-3, max_iter=6)
    out = []
    for rows in (0, 1, 2, 4):
        ps = [p] if rows == 0 else [p, tdgl.make_params(256, 256, 17, bc=(1, 1, 1), tol=1e6, max_iter=6)]
        s = tdgl.Solver(ps)    # alone: blocks; beside a large box: single sweeps
        if rows:
            s.set_tiling(rows=rows)
        s.set_field(0.0, 0.1, inst=0)
        s.set_psi(torch.from_numpy(psi).cuda(), inst=0)
        st = s.step(1)
        assert st["capped_steps"] == 1 and st["sweeps_max"] == 6
        out.append(s.get_psi(0).cpu().numpy())
        s.close()
    assert np.isnan(out[0]).any() and not np.isnan(out[0]).all()
    for o in out[1:]:
        assert np.array_equal(out[0], o, equal_nan=True)
