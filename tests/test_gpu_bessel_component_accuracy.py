"""Each field component of the Bessel form's contraction against the FP64 oracle in its own norm, at
apertures where I_1 and I_2 are orders of magnitude below I_0, and the gradient there."""
import numpy as np
import pytest

from oracle import adjoint_bessel as AB
from oracle import bessel as OB
from oracle import optics as O
from oracle.adjoint import mse_loss
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu
# FP32's level: a sum of 128 terms whose roundings (2^-24 each) do not add up and an interpolation of four
# samples, under eight of them
TOL = 8 * 2.0 ** -24


@pytest.mark.parametrize("na", [0.003, 0.005, 0.02, 0.1, 1.4])
@pytest.mark.parametrize("e_inc", [(1.0, 0.0), (0.0, 1j), (1.0, 1e-6)])
@pytest.mark.parametrize("n_stacks", [2, 80])   # 64-column and 256-column tiles
def test_components(lib, na, e_inc, n_stacks):
    pixel = 30.0 / na
    z = np.linspace(-200.0, 300.0, 66) / na ** 2
    zernike = np.zeros(22)
    zernike[3], zernike[10] = 0.06, -0.04
    plan = lib.Plan(form=lib.FORM_BESSEL, na=na, wavelength=532.0, n_i=1.518, nx=24, ny=20, dx=pixel, dy=pixel, z=z,
                    e_inc=e_inc, n_theta=128, n_rho=512)
    E = plan.compute([dict(zernike=zernike)] * n_stacks)[0][n_stacks - 1].cpu().numpy()
    plan.close()
    opt = O.Optics(na=na, wavelength=532.0, n_i=1.518, e_inc=e_inc)
    ref = OB.field_bessel(opt, 24, 20, pixel, pixel, z, n_theta=128, zernike=zernike)
    for c in range(3):
        assert rel_l2(E[:, c], ref[:, c]) < TOL


@pytest.mark.parametrize("na", [0.005, 0.1])
@pytest.mark.parametrize("fields", [(1, 1, 1), (0, 1, 0), (0, 0, 1)])   # components that the loss looks at
def test_gradient_of_weak_components(lib, na, fields):
    """The gradient of a loss that has only the weak components' light (the others' fields are zero), in the
    coefficients without piston (piston and, at these apertures, defocus change next to nothing)."""
    import torch
    pixel = 30.0 / na
    z = np.linspace(-200.0, 300.0, 5) / na ** 2
    coeffs = np.zeros(22)
    coeffs[3], coeffs[10] = 0.06, -0.04
    stacks = [(0.0, 0.1 * pixel, -0.2 * pixel, 60.0 / na ** 2)]
    plan = lib.Plan(form=lib.FORM_BESSEL, na=na, wavelength=532.0, n_i=1.518, nx=24, ny=20, dx=pixel, dy=pixel, z=z,
                    e_inc=(1.0, 0.0), n_theta=128, n_rho=512)
    opt = O.Optics(na=na, wavelength=532.0, n_i=1.518, e_inc=(1.0, 0.0))
    keep = np.array(fields, dtype=np.float64)[None, None, :, None, None]
    E, _ = AB.forward(opt, 24, 20, pixel, pixel, z, coeffs, stacks, 128)
    I = (np.abs(E * keep) ** 2).sum(axis=2)
    rng = np.random.default_rng(4)
    g = mse_loss(I, I * (0.7 + 0.2 * rng.standard_normal(I.shape)) / I.max(), np.array([1.0 / I.max()]))[1]
    st = [dict(x0=s[1], y0=s[2], z_offset=s[3], zernike=coeffs) for s in stacks]
    Et = torch.tensor((E * keep).astype(np.complex64), device="cuda")
    dc = plan.adjoint_bessel(st, Et, torch.tensor(g, dtype=torch.float32, device="cuda"))[0]
    torch.cuda.synchronize()
    plan.close()
    # the oracle's gradient is linear in the fields that it pulls back
    forward = AB.forward
    try:
        AB.forward = lambda *a, **k: (E * keep, None)
        rdc = AB.gradient(opt, 24, 20, pixel, pixel, z, coeffs, stacks, g, 128)[0]
    finally:
        AB.forward = forward
    assert rel_l2(dc.double().cpu().numpy()[1:], rdc[1:]) < 1e-5
