"""Column pass of the chirp-z form against the FP64 oracle: 16, 8 and 4 columns a workgroup with a
last block of fewer, more inputs than outputs and the reverse, one channel and three, and the
longest output whose padded columns do not fit LDS."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_fourier_stack, oracle_optics, rel_l2

pytestmark = pytest.mark.gpu
TOL = 1e-5   # the bar of the FP32 forms


@pytest.mark.parametrize("n_pupil,nx,ny", [
    (256, 128, 17), (40, 200, 35), (30, 20, 50), (400, 100, 11), (100, 390, 9), (900, 100, 6), (20, 1000, 5),
    (2, 1875, 3)])
def test_chirpz_column_blocks(lib, n_pupil, nx, ny):
    import torch
    rw = lib
    w = W.fourier_plain(n_stacks=1, seed=7)
    z = np.array([-300.0, 400.0])
    o = w["optics"]
    plan = rw.Plan(form=rw.FORM_CHIRPZ, na=o["na"], wavelength=o["wavelength"], n_i=o["n_i"], nx=nx, ny=ny, dx=15.0,
                   dy=15.0, z=z, e_inc=w["e_inc"], n_pupil=n_pupil)
    E, I = plan.compute([dict(x0=9.0, y0=-5.0, zernike=w["zernike"][0])])
    torch.cuda.synchronize()
    plan.close()
    ref = oracle_fourier_stack(oracle_optics(w, gl=False), n_pupil, nx, ny, 15.0, 15.0, z, zernike=w["zernike"][0],
                               x0=9.0, y0=-5.0)
    assert rel_l2(E[0].cpu().numpy(), ref) < TOL
    assert rel_l2(I[0].cpu().numpy(), (np.abs(ref) ** 2).sum(axis=1)) < TOL


@pytest.mark.parametrize("n_pupil,nx,ny,nz", [(40, 30, 33, 90), (60, 24, 17, 129), (300, 260, 35, 90)])
def test_chirpz_column_blocks_of_few_and_many_planes(lib, n_pupil, nx, ny, nz):
    """A call of few planes takes fewer columns a workgroup; a plane does not depend on it."""
    rw = lib
    w = W.fourier_plain(n_stacks=1, seed=8)
    z = np.linspace(-500.0, 500.0, nz)
    o = w["optics"]
    st = [dict(x0=9.0, y0=-5.0, zernike=w["zernike"][0])]

    def fields(zz):
        plan = rw.Plan(form=rw.FORM_CHIRPZ, na=o["na"], wavelength=o["wavelength"], n_i=o["n_i"], nx=nx, ny=ny,
                       dx=15.0, dy=15.0, z=zz, e_inc=w["e_inc"], n_pupil=n_pupil)
        E, I = plan.compute(st)
        E, I = E[0].cpu().numpy(), I[0].cpu().numpy()
        plan.close()
        return E, I

    E, I = fields(z)
    E1, I1 = fields(z[:1])
    assert np.array_equal(E[:1], E1) and np.array_equal(I[:1], I1)
    En, In = fields(z[-3:])
    assert np.array_equal(E[-3:], En) and np.array_equal(I[-3:], In)
