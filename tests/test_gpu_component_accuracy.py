"""Each field component against the FP64 oracle in its own norm, at apertures where the longitudinal and
cross-polarised components are orders of magnitude smaller than the main one."""
import numpy as np
import pytest

from oracle import fourier as OF
from oracle import optics as O
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu
# FP32's level: sums of many terms whose roundings (2^-24 each) do not add up, under five of them
TOL = 5 * 2.0 ** -24
POL = [(1.0, 0.0), (0.0, 1j), (1.0, 1e-6)]


def _setting(na):
    pixel = 30.0 / na
    zernike = np.zeros(21)
    zernike[4], zernike[6], zernike[9] = 0.06, -0.05, 0.04
    return pixel, zernike


def _reference(n, na, e_inc, nx, ny, pixel, z, zernike):
    opt = O.Optics(na=na, wavelength=532.0, n_i=1.518, e_inc=e_inc)
    g = OF.pupil_geometry(n, opt)
    return OF.field_separable(OF.base_pupil(g, opt, OF.pupil_phase(g, opt, zernike=zernike)), g, opt, nx, ny, pixel, pixel, z)


@pytest.mark.parametrize("na", [0.005, 0.02, 0.1, 1.4])
@pytest.mark.parametrize("e_inc", POL)
@pytest.mark.parametrize("n,nx,ny,nz,n_stacks", [(64, 48, 40, 4, 1), (64, 70, 66, 3, 1), (64, 64, 64, 19, 9), (50, 130, 130, 19, 9)])
def test_fourier_components(lib, na, e_inc, n, nx, ny, nz, n_stacks):
    import torch
    pixel, zernike = _setting(na)
    z = np.linspace(-200.0, 300.0, nz) / na ** 2
    plan = lib.Plan(form=lib.FORM_FOURIER, na=na, wavelength=532.0, n_i=1.518, nx=nx, ny=ny, dx=pixel, dy=pixel, z=z,
                    e_inc=e_inc, n_pupil=n)
    E = plan.compute([dict(zernike=zernike)] * n_stacks)[0][n_stacks - 1].cpu().numpy()
    plan.close()
    ref = _reference(n, na, e_inc, nx, ny, pixel, z, zernike)
    for c in range(3):
        assert rel_l2(E[:, c], ref[:, c]) < TOL


@pytest.mark.parametrize("na", [0.005, 0.02, 1.4])
@pytest.mark.parametrize("e_inc", POL)
@pytest.mark.parametrize("n", [32, 64, 96, 128])
@pytest.mark.parametrize("crop", [31, 64])
def test_batch_components(lib, na, e_inc, n, crop):
    import torch
    pixel, zernike = _setting(na)
    pitch = 50.0 / na ** 2
    batch = lib.Batch(na=na, wavelength=532.0, n_i=1.518, pixel=pixel, plane_pitch=pitch, max_emitters=1, n_pupil=n,
                      e_inc=e_inc)
    E = torch.empty(3 * 2 * crop * crop, dtype=torch.complex64, device="cuda")
    batch.compute(lib.make_emitters([0.0], [0.0], [0.0], [crop], [2], zernike[None]), None, E)
    E = E.view(2, 3, crop, crop).cpu().numpy()
    batch.close()
    ref = _reference(n, na, e_inc, crop, crop, pixel, np.array([-0.5, 0.5]) * pitch, zernike)
    for c in range(3):
        assert rel_l2(E[:, c], ref[:, c]) < TOL
