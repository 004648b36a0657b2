"""Few image tiles (channels side by side in a workgroup) and just too many for that: the FP64
oracle, three channels and one, fields or intensity only, ragged and whole tiles."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_fourier_stack, oracle_optics, rel_l2

pytestmark = pytest.mark.gpu
TOL = 1e-5   # the bar of the FP32 forms


# tiles of 32 x 64 pixels, padded to 64 (128 above 64): planes x tiles below and above 256 CUs
@pytest.mark.parametrize("n_pupil,nx,ny,nz", [(40, 1, 1, 1), (65, 64, 64, 3), (96, 201, 130, 1), (64, 65, 64, 32),
                                              (64, 64, 64, 129), (33, 130, 70, 9)])
@pytest.mark.parametrize("fields,intensity", [(True, True), (True, False), (False, True)])
def test_fourier_few_tiles(lib, n_pupil, nx, ny, nz, fields, intensity):
    import torch
    rw = lib
    w = W.fourier_plain(n_stacks=1, seed=3)
    z = np.linspace(-300.0, 200.0, nz)
    plan = rw.Plan(form=rw.FORM_FOURIER, **w["optics"], nx=nx, ny=ny, dx=30.0, dy=30.0, z=z, e_inc=w["e_inc"],
                   n_pupil=n_pupil)
    E = torch.zeros(nz, 3, nx, ny, dtype=torch.complex64, device="cuda") if fields else None
    I = torch.zeros(nz, nx, ny, dtype=torch.float32, device="cuda") if intensity else None
    rw.compute(plan, [dict(x0=5.0, zernike=w["zernike"][0])], E, I)
    torch.cuda.synchronize()
    plan.close()
    ref = oracle_fourier_stack(oracle_optics(dict(w, gl=None)), n_pupil, nx, ny, 30.0, 30.0, z, x0=5.0,
                               zernike=w["zernike"][0])
    if fields:
        assert rel_l2(E.cpu().numpy(), ref) < TOL
    if intensity:
        assert rel_l2(I.cpu().numpy(), (np.abs(ref) ** 2).sum(axis=1)) < TOL


def test_fourier_few_tiles_scalar(lib):
    import torch
    rw = lib
    z = np.array([0.0, 250.0])
    common = dict(na=1.2, wavelength=500.0, n_i=1.33, nx=50, ny=90, dx=40.0, dy=40.0, z=z, n_pupil=64)
    plan = rw.Plan(form=rw.FORM_FOURIER, model=rw.MODEL_SCALAR, **common)
    E, I = plan.compute([dict()])
    many, Im = plan.compute([dict()] * 200)
    torch.cuda.synchronize()
    plan.close()
    assert rel_l2(E[0].cpu().numpy(), many[57].cpu().numpy()) < 1e-6
    assert rel_l2(I[0].cpu().numpy(), (E[0].abs() ** 2).sum(1).cpu().numpy()) < 1e-6
