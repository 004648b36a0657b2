"""Gradients of fields and dL/dI that start anywhere in a larger tensor equal those of tensors of
their own."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(32, 48), (48, 80)])   # one and two chunks along y
@pytest.mark.parametrize("e_at,g_at", [(1, 0), (0, 1), (0, 2), (1, 3)])
def test_views(lib, nx, ny, e_at, g_at):
    import torch
    rw = lib
    w = W.fourier_plain(n_stacks=2, seed=3)
    plan = rw.Plan(form=rw.FORM_FOURIER, **w["optics"], nx=nx, ny=ny, dx=100.0, dy=100.0, z=np.linspace(-300.0, 300.0, 3),
                   e_inc=w["e_inc"], n_pupil=64)
    st = [dict(x0=9.0 * b, z_offset=30.0 * b, zernike=w["zernike"][b]) for b in range(2)]
    E, I = plan.compute(st)
    g = I - 0.3 * I.max()
    ref = plan.adjoint(st, E, g, 21)
    Ev = torch.empty(E.numel() + 4, dtype=E.dtype, device="cuda")[e_at:e_at + E.numel()].view(E.shape)
    gv = torch.empty(g.numel() + 4, device="cuda")[g_at:g_at + g.numel()].view(g.shape)
    Ev.copy_(E)
    gv.copy_(g)
    got = plan.adjoint(st, Ev, gv, 21)
    torch.cuda.synchronize()
    plan.close()
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
