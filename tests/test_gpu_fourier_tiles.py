"""Tile classes of the Fourier form's two GEMMs against the FP64 oracle: launches large enough
for the tall tiles (two planes a tile; an odd plane count leaves half a tile), outputs of at
most and of more than 64 pixels along each axis, rows that allow wide stores and rows that
do not, and pupils of very small amplitude (the operand scales)."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_fourier_stack, oracle_optics, rel_l2

pytestmark = pytest.mark.gpu
TOL = 1e-5   # the bar of the FP32 forms


# (pupil, nx, ny, nz, stacks): 3 nz stacks >= 512 tiles of 128 rows takes the tall tiles
@pytest.mark.parametrize("n_pupil,nx,ny,nz,n_stacks,na", [
    (64, 33, 64, 19, 9, 1.4), (50, 65, 31, 43, 4, 1.4), (64, 128, 130, 19, 9, 1.4), (97, 70, 65, 9, 11, 1.4),
    (64, 40, 66, 1, 1, 1.4), (64, 64, 64, 19, 9, 0.02)])
@pytest.mark.parametrize("offset", [0, 1])   # 1: outputs that do not allow wide stores
def test_fourier_tile_classes(lib, n_pupil, nx, ny, nz, n_stacks, na, offset):
    import torch
    rw = lib
    w = W.fourier_plain(n_stacks=n_stacks, seed=5)
    w["optics"] = dict(w["optics"], na=na)
    z = np.linspace(-500.0, 700.0, nz)
    plan = rw.Plan(form=rw.FORM_FOURIER, **w["optics"], nx=nx, ny=ny, dx=30.0, dy=30.0, z=z, e_inc=w["e_inc"],
                   n_pupil=n_pupil)
    stacks = [dict(x0=7.0 * b, y0=-4.0 * b, z_offset=11.0 * b, zernike=w["zernike"][b]) for b in range(n_stacks)]
    vox = n_stacks * nz * nx * ny
    E = torch.zeros(3 * vox + 2, dtype=torch.complex64, device="cuda")
    I = torch.zeros(vox + 2, dtype=torch.float32, device="cuda")
    rw.compute(plan, stacks, E[offset:], I[offset:])
    torch.cuda.synchronize()
    plan.close()
    assert not (E[3 * vox + offset:].any() or E[:offset].any() or I[vox + offset:].any() or I[:offset].any())
    e = E[offset:offset + 3 * vox].view(n_stacks, nz, 3, nx, ny).cpu().numpy()
    i = I[offset:offset + vox].view(n_stacks, nz, nx, ny).cpu().numpy()
    opt = oracle_optics(dict(w, gl=None))
    for b in sorted({0, n_stacks // 2, n_stacks - 1}):
        s = stacks[b]
        ref = oracle_fourier_stack(opt, n_pupil, nx, ny, 30.0, 30.0, z + s["z_offset"], zernike=s["zernike"],
                                   x0=s["x0"], y0=s["y0"])
        assert rel_l2(e[b], ref) < TOL
        assert rel_l2(i[b], (np.abs(ref) ** 2).sum(axis=1)) < TOL
