"""A gradient call that runs out of memory while it builds its workspace fails each time it is made, and
the same plan gives the right gradient once there is room."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _fill(left):
    """Tensors that leave between `left` and `left` + 128 MB of the device's memory."""
    import torch
    hogs = []
    while (free := torch.cuda.mem_get_info()[0]) > left + (1 << 27):
        try:
            hogs.append(torch.empty(min(free - left, 32 << 30), dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:
            break
    return hogs


def test_bessel_adjoint_after_out_of_memory(lib):
    import torch
    rw = lib
    w = W.bessel_plain()
    kw = dict(form=rw.FORM_BESSEL, na=1.4, wavelength=532.0, n_i=1.518, nx=5, ny=5, dx=20.0, dy=20.0,
              z=np.linspace(-300.0, 300.0, 129), e_inc=w["e_inc"], n_theta=64, n_rho=2048)
    st = [dict(z_offset=40.0)]
    plan, other = rw.Plan(**kw), rw.Plan(**kw)
    E, I = plan.compute(st)
    ref = other.adjoint_bessel(st, E, I)
    torch.cuda.synchronize()
    other.close()   # its 0.5 GB of workspace and 1.7 GB of scratch are free again
    hogs = _fill(1 << 28)   # less than the 0.4 GB of the radial samples' gradients
    for _ in range(2):
        with pytest.raises(rw.RwpsfError) as ei:
            plan.adjoint_bessel(st, E, I)
        assert ei.value.status == rw.ERR_OOM
    del hogs
    torch.cuda.empty_cache()
    got = plan.adjoint_bessel(st, E, I)
    torch.cuda.synchronize()
    plan.close()
    for a, b in zip(got, ref):
        assert torch.equal(a, b)


def test_fourier_adjoint_after_out_of_memory(lib):
    """A retry does not allocate again what the failed call had."""
    import torch
    rw = lib
    w = W.fourier_plain(n_stacks=1, seed=3)
    kw = dict(form=rw.FORM_FOURIER, **w["optics"], nx=16, ny=16, dx=100.0, dy=100.0, z=np.linspace(-300.0, 300.0, 9),
              e_inc=w["e_inc"], n_pupil=512)
    st = [dict(zernike=w["zernike"][0])] * 64
    plan, other = rw.Plan(**kw), rw.Plan(**kw)
    E, I = plan.compute(st)
    ref = other.adjoint(st, E, I, 21)
    torch.cuda.synchronize()
    other.close()   # the pupils of a launch take 0.4 GB, the partial sums of 64 stacks 0.2 GB or more
    hogs = _fill((1 << 28) + (1 << 27) + (1 << 26))
    held = []
    for _ in range(3):
        with pytest.raises(rw.RwpsfError) as ei:
            plan.adjoint(st, E, I, 21)
        assert ei.value.status == rw.ERR_OOM
        held.append(plan.device_bytes())
    assert held[0] == held[2]
    del hogs
    torch.cuda.empty_cache()
    got = plan.adjoint(st, E, I, 21)
    torch.cuda.synchronize()
    plan.close()
    for a, b in zip(got, ref):
        assert torch.equal(a, b)
