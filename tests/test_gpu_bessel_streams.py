"""Bessel-form calls whose fields leave the last-level cache (256 MB) run the epilogue with neighbouring
planes on one XCD and fewer workgroups a CU: bit for bit the results of smaller calls."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# 28 B a pixel (12 in the scalar model): past 256 MB in all, below it in parts; planes of fewer and of more
# than 2048 pixels, counts of planes that are no multiple of the XCDs
@pytest.mark.parametrize("nx,ny,nz,n_stacks,kind", [
    (65, 65, 33, 69, "vectorial"), (33, 31, 51, 190, "fresnel"), (61, 67, 33, 171, "scalar"), (64, 64, 33, 71, "vectorial")])
def test_large_call_equals_smaller_calls(lib, nx, ny, nz, n_stacks, kind):
    import torch
    rw = lib
    w = W.bessel_plain()
    plan = rw.Plan(form=rw.FORM_BESSEL, na=1.4, wavelength=532.0, n_i=1.518, nx=nx, ny=ny, dx=20.0, dy=20.0,
                   z=np.linspace(-600.0, 600.0, nz), e_inc=w["e_inc"], n_theta=128, n_rho=160,
                   fresnel=(1.33, 1.5) if kind == "fresnel" else None,
                   model=rw.MODEL_SCALAR if kind == "scalar" else rw.MODEL_VECTORIAL)
    rng = np.random.default_rng(nz)
    st = [dict(x0=rng.uniform(-15, 15), y0=rng.uniform(-15, 15), z_offset=rng.uniform(-100, 100)) for _ in range(n_stacks)]
    E, I = plan.compute(st)
    assert E.numel() * 8 + I.numel() * 4 > 256 << 20
    for b in range(0, n_stacks, 32):
        e, i = plan.compute(st[b:b + 32])
        assert torch.equal(E[b:b + 32], e) and torch.equal(I[b:b + 32], i)
    only, _ = plan.compute(st, intensity=False)
    assert torch.equal(only, E)
    plan.close()
