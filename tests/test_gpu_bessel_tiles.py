"""Bessel form: the contraction's two tiles at row, column and node counts beside their edges, planes
of fewer and of more pixels than the adjoint keeps in registers, and the operand exponents."""
import numpy as np
import pytest

import workloads as W
from oracle import bessel as OB
from oracle import optics as O
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu
TOL = 1e-5   # the bar of the FP32 forms


# rows 2 stacks nz: 64-column tiles below 256 tiles of 64 x 256, else those; nodes around multiples of
# 16 and of the 128 that a run keeps, columns 3 rho around multiples of 64
@pytest.mark.parametrize("nx,nz,n_stacks,n_theta,n_rho", [
    (9, 5, 13, 128, 64), (9, 16, 4, 129, 170), (7, 33, 130, 145, 171), (5, 64, 128, 127, 257)])
def test_bessel_contract_tiles(lib, nx, nz, n_stacks, n_theta, n_rho):
    import torch
    rw = lib
    w = W.bessel_plain()
    z = np.linspace(-600.0, 600.0, nz)
    plan = rw.Plan(form=rw.FORM_BESSEL, na=1.4, wavelength=532.0, n_i=1.518, nx=nx, ny=nx + 2, dx=20.0, dy=20.0, z=z,
                   e_inc=w["e_inc"], n_theta=n_theta, n_rho=n_rho)
    rng = np.random.default_rng(nz)
    st = [dict(x0=rng.uniform(-15, 15), y0=rng.uniform(-15, 15), z_offset=rng.uniform(-100, 100)) for _ in range(n_stacks)]
    E, I = plan.compute(st)
    torch.cuda.synchronize()
    plan.close()
    opt = O.Optics(na=1.4, wavelength=532.0, n_i=1.518, e_inc=w["e_inc"])
    for b in (0, n_stacks // 2, n_stacks - 1):
        s = st[b]
        ref = OB.field_bessel(opt, nx, nx + 2, 20.0, 20.0, z + s["z_offset"], x0=s["x0"], y0=s["y0"], n_theta=256)
        assert rel_l2(E[b].cpu().numpy(), ref) < TOL
        assert rel_l2(I[b].cpu().numpy(), (np.abs(ref) ** 2).sum(axis=1)) < TOL


@pytest.mark.parametrize("nx,ny", [(16, 32), (67, 69), (48, 96), (71, 73)])   # 512 threads x 9 pixels = 4608
def test_bessel_adjoint_planes_and_scales(lib, nx, ny):
    """Exactly linear in powers of two of dL/dI, planes without gradient among others, and equal to the
    sum over calls of one stack."""
    import torch
    rw = lib
    w = W.bessel_plain()
    z = np.linspace(-400.0, 400.0, 3)
    plan = rw.Plan(form=rw.FORM_BESSEL, na=1.4, wavelength=532.0, n_i=1.518, nx=nx, ny=ny, dx=20.0, dy=20.0, z=z,
                   e_inc=w["e_inc"], n_theta=150, n_rho=160)
    st = [dict(x0=3.0, y0=-8.0, z_offset=40.0), dict(x0=-11.0, y0=5.0, z_offset=-90.0)]
    E, I = plan.compute(st)
    g = (I - 0.3 * I.max()).contiguous()
    g[0, 1] = 0.0
    dc, dts, dz = plan.adjoint_bessel(st, E, g)
    for e in (-30, 20):
        c2, _, z2 = plan.adjoint_bessel(st, E, g * 2.0 ** e)
        assert torch.equal(c2, dc * 2.0 ** e) and torch.equal(z2, dz * 2.0 ** e)
    parts = [plan.adjoint_bessel(st[i:i + 1], E[i:i + 1].contiguous(), g[i:i + 1].contiguous()) for i in (0, 1)]
    torch.cuda.synchronize()
    assert rel_l2((parts[0][0] + parts[1][0]).cpu().numpy(), dc.cpu().numpy()) < TOL
    assert torch.equal(torch.cat([parts[0][2], parts[1][2]]), dz)
    plan.close()
