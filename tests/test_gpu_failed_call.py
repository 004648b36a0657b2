"""A call that fails leaves nothing behind: the next call of another handle succeeds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _too_large_plan(rw):
    # radial samples of 256 stacks of 16384 planes: about 1 TB
    rw.Plan(form=rw.FORM_BESSEL, na=1.4, wavelength=532.0, n_i=1.518, nx=4, ny=4, dx=20.0, dy=20.0,
            z=np.linspace(-9.0, 9.0, 16384), n_theta=16, n_rho=3000, fresnel=(1.33, 1.5))


def _too_large_batch(rw):
    # folded pupils of 2^20 emitters: 412 GB
    rw.Batch(na=1.4, wavelength=532.0, n_i=1.518, pixel=100.0, plane_pitch=50.0, max_emitters=1 << 20)


@pytest.mark.parametrize("fail", [_too_large_plan, _too_large_batch])
@pytest.mark.parametrize("form", ["FORM_BESSEL", "FORM_FOURIER", "FORM_CHIRPZ"])
def test_call_after_out_of_memory(lib, fail, form):
    import torch
    rw = lib
    plan = rw.Plan(form=getattr(rw, form), na=1.4, wavelength=532.0, n_i=1.518, nx=8, ny=8, dx=20.0, dy=20.0, z=[0.0],
                   n_pupil=32, n_theta=32, n_rho=32)
    ref = plan.compute([dict()])[1].clone()
    with pytest.raises(rw.RwpsfError) as ei:
        fail(rw)
    assert ei.value.status == rw.ERR_OOM
    got = plan.compute([dict()])[1]
    torch.cuda.synchronize()
    plan.close()
    assert torch.equal(got, ref)
