"""Workspace of the Fourier form's gradient: bounded in the stacks of a call and in the image's width,
no growth for a smaller call after a larger one, and results that do not depend on how a call is split
into launches."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu
GIB = 1 << 30


def _plan(rw, n_pupil, nx, ny, nz):
    w = W.fourier_plain(n_stacks=1, seed=3)
    return rw.Plan(form=rw.FORM_FOURIER, **w["optics"], nx=nx, ny=ny, dx=100.0, dy=100.0,
                   z=np.linspace(-300.0, 300.0, nz), e_inc=w["e_inc"], n_pupil=n_pupil)


def _stacks(n):
    rng = np.random.default_rng(n)
    return [dict(x0=rng.uniform(-50, 50), y0=rng.uniform(-50, 50), z_offset=rng.uniform(-200, 200),
                 zernike=rng.normal(0, 0.03, 21)) for _ in range(n)]


def _sum_of_parts(plan, st, E, g, per):
    dc, dw = 0.0, 0.0
    for i in range(0, len(st), per):
        c, w = plan.adjoint(st[i:i + per], E[i:i + per].contiguous(), g[i:i + per].contiguous(), 21)
        dc, dw = dc + c.double().cpu().numpy(), dw + w.double().cpu().numpy()
    return dc, dw


def test_more_stacks_than_a_launch(lib):
    plan = _plan(lib, 512, 16, 16, 1)
    st = _stacks(300)
    E, I = plan.compute(st)
    g = I - 0.3 * I.max()
    ref = _sum_of_parts(plan, st, E, g, 64)
    before = plan.device_bytes()
    dc, dw = plan.adjoint(st, E, g, 21)
    assert plan.device_bytes() - before < 1 << 20   # scales of the planes, nothing else
    assert rel_l2(dc.double().cpu().numpy(), ref[0]) < 1e-6 and rel_l2(dw.double().cpu().numpy(), ref[1]) < 1e-6
    plan.close()


def test_wide_image_and_large_pupil(lib):
    plan = _plan(lib, 1024, 512, 16, 3)
    st = _stacks(33)
    E, I = plan.compute(st)
    g = I - 0.3 * I.max()
    before = plan.device_bytes()
    dc, dw = plan.adjoint(st, E, g, 21)
    # 1.6 GB of folded pupils, 1 GiB of partial sums and a sixteenth of it of their runs
    assert plan.device_bytes() - before < 3 * GIB
    ref = _sum_of_parts(plan, st, E, g, 1)
    # FP32 sums over runs of other lengths
    assert rel_l2(dc.double().cpu().numpy(), ref[0]) < 1e-5 and rel_l2(dw.double().cpu().numpy(), ref[1]) < 1e-5
    plan.close()


@pytest.mark.parametrize("nx,ny", [(64, 64), (80, 144)])
def test_smaller_call_after_a_larger_one(lib, nx, ny):
    plan = _plan(lib, 64, nx, ny, 21)
    st = _stacks(64)
    E, I = plan.compute(st)
    plan.adjoint(st, E, I, 21)
    before = plan.device_bytes()
    for n in range(1, 64):
        plan.adjoint(st[:n], E[:n], I[:n], 21)
    assert plan.device_bytes() == before
    plan.close()
