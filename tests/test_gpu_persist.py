"""Persistent Jacobi solves whose grid fills the chip: every work-group has to
be resident at once, so the grid may not exceed what fits."""
import numpy as np
import pytest

from paper_1409_8340_amd import inputs, tdgl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,rows,chunk", [
    ((288, 270, 19), 1, 4),   # 1700 tiles: more than six work-groups per CU
    ((288, 270, 19), 2, 4),
    ((320, 256, 24), 4, 2),
])
def test_persistent_grid_fits(shape, rows, chunk):
    # the same node arithmetic in another order of work: equal bits
    import torch
    nx, ny, nz = shape
    psi = torch.from_numpy(inputs.random_complex((nz, ny, nx), 5, 0.5).astype(np.complex64)).cuda()
    out = []
    for persist in (0, 1):
        p = tdgl.make_params(nx, ny, nz, max_iter=40, tol=1e-10)
        s = tdgl.Solver(p)
        s.set_field(0.03, 0.2, quantize=True)
        s.set_tiling(rows=rows, chunk=chunk, persistent=persist)
        s.set_psi(psi)
        st = s.step(2)
        out.append((s.get_psi().cpu(), st["sweeps_sum"]))
        s.close()
    assert out[0][1] == out[1][1]
    assert torch.equal(torch.view_as_real(out[0][0]), torch.view_as_real(out[1][0]))
