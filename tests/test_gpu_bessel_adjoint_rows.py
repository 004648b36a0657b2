"""Bessel-form adjoint against the FP64 gradient oracle for counts of radial samples whose rows are no
multiple of a wide load, and at a size that takes the contraction's wide tiles."""
import numpy as np
import pytest

import workloads as W
from oracle import adjoint_bessel as AB
from oracle import optics as O
from oracle.adjoint import mse_loss
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu
TOL = 1e-5   # the bar of the FP32 forms


def _check(rw, kind, nx, ny, z, n_stacks, n_theta, n_rho):
    import torch
    GL = W.GIBSON_LANNI
    scalar, media = kind == "scalar", (GL["n_s"], GL["n_g"]) if kind == "fresnel" else None
    dx = 40.0
    plan = rw.Plan(form=rw.FORM_BESSEL, na=1.4, wavelength=600.0, n_i=1.518, nx=nx, ny=ny, dx=dx, dy=dx, z=z,
                   e_inc=W.CIRCULAR, gibson_lanni=dict(GL), n_theta=n_theta, n_rho=n_rho,
                   model=rw.MODEL_SCALAR if scalar else rw.MODEL_VECTORIAL, fresnel=media)
    gl = O.GibsonLanni(n_s=GL["n_s"], n_g=GL["n_g"], n_g_design=GL["n_g_design"], n_i_design=GL["n_i_design"],
                       t_g=GL["t_g"], t_g_design=GL["t_g_design"], t_i_design=GL["t_i_design"])
    opt = O.Optics(na=1.4, wavelength=600.0, n_i=1.518, e_inc=W.CIRCULAR, gl=gl, fresnel_media=media or ())
    rng = np.random.default_rng(n_rho)
    coeffs = np.zeros(22)
    coeffs[3], coeffs[10], coeffs[21] = 0.05, -0.04, 0.03
    ts = rng.uniform(500.0, 3000.0, n_stacks)
    stacks = [(float(t), float(rng.uniform(-15, 15)), float(rng.uniform(-15, 15)), float(-t + rng.uniform(-200, 200)))
              for t in ts]
    args = (nx, ny, dx, dx, z)
    _, I0 = AB.forward(opt, *args, coeffs, stacks, 256, "gauss", scalar)
    c2 = coeffs.copy()
    c2[3] += 0.03
    _, I1 = AB.forward(opt, *args, c2, stacks, 256, "gauss", scalar)
    scale = (1.0 + 0.1 * (np.arange(n_stacks) % 7)) / I0.max()
    Y = scale[:, None, None, None] * I1 * (1 + 0.2 * rng.standard_normal(I1.shape))
    g = mse_loss(I0, Y, scale)[1]
    st = [dict(t_s=s[0], x0=s[1], y0=s[2], z_offset=s[3], zernike=coeffs) for s in stacks]
    E, _ = plan.compute(st, intensity=False)
    got = plan.adjoint_bessel(st, E, torch.tensor(g, dtype=torch.float32, device="cuda"))
    torch.cuda.synchronize()
    plan.close()
    dc, dts, dz = (x.double().cpu().numpy() for x in got)
    rdc, rdts, rdz = AB.gradient(opt, *args, coeffs, stacks, g, 256, "gauss", scalar)
    assert rel_l2(dc[1:], rdc[1:]) < TOL and rel_l2(dts, rdts) < TOL and rel_l2(dz, rdz) < TOL


# columns 3 rho, 5 rho or rho: odd, twice an odd number, a last run of fewer than eight
@pytest.mark.parametrize("kind", ["vectorial", "fresnel", "scalar"])
@pytest.mark.parametrize("n_rho", [161, 171, 174])
def test_rows_of_any_length(lib, kind, n_rho):
    _check(lib, kind, 17, 15, np.array([-400.0, 0.0, 350.0]), 2, 400, n_rho)


# 2 64 64 rows and more than 256 nodes: 256 tiles of 64 x 256 or more
@pytest.mark.parametrize("kind,n_rho", [("vectorial", 163), ("fresnel", 160), ("scalar", 169)])
def test_wide_tiles(lib, kind, n_rho):
    _check(lib, kind, 7, 6, np.linspace(-500.0, 450.0, 64), 64, 400, n_rho)
