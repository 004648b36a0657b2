"""Bessel-form adjoint of gradients and fields that hold a NaN or an infinity: the stack that has it
gets NaN, every other stack what it gets without."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
KINDS = {"vectorial": {}, "fresnel": dict(fresnel=(1.33, 1.5)), "scalar": dict()}


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("nx,pixel", [(9, 0), (9, 80), (71, 70 * 73)])   # kept in registers, read again
def test_not_finite_pixel(lib, kind, nx, pixel):
    import torch
    rw = lib
    w = W.bessel_plain()
    z = np.linspace(-300.0, 300.0, 3)
    plan = rw.Plan(form=rw.FORM_BESSEL, na=1.4, wavelength=532.0, n_i=1.518, nx=nx, ny=nx + 2, dx=20.0, dy=20.0, z=z,
                   e_inc=w["e_inc"], gibson_lanni=dict(W.GIBSON_LANNI), n_theta=96, n_rho=160,
                   model=rw.MODEL_SCALAR if kind == "scalar" else rw.MODEL_VECTORIAL, **KINDS[kind])
    st = [dict(t_s=900.0, z_offset=-900.0 + 30.0 * b, x0=2.0 * b) for b in range(3)]
    E, I = plan.compute(st)
    g = (I - 0.3 * I.max()).contiguous()
    ref = plan.adjoint_bessel(st, E, g)
    i, j = divmod(pixel, nx + 2)
    only = torch.zeros_like(g)   # the pixel is the stack's only gradient
    only[0], only[2] = g[0], g[2]
    for rest in (g, only):
        for bad in (float("nan"), float("inf")):
            g2, E2 = rest.clone(), E.clone()
            g2[1, 2, i, j] = bad
            E2[1, 2, 0, i, j] = complex(bad, 0.0)
            cases = [(E, g2)] + ([(E2, rest)] if rest is g else [])
            for e, h in cases:
                dc, dts, dz = plan.adjoint_bessel(st, e, h)
                torch.cuda.synchronize()
                assert torch.isnan(dz[1]) and torch.isnan(dts[1]) and torch.isnan(dc).all()
                for b in (0, 2):
                    assert torch.equal(dz[b], ref[2][b]) and torch.equal(dts[b], ref[1][b])
    plan.close()
