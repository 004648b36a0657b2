"""A gradient call that runs out of memory while it builds its workspace fails each time it is made, and
the same plan gives the right gradient once there is room."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


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
    # leave less than the 0.4 GB of the radial samples' gradients
    hogs, left = [], 1 << 28
    while (free := torch.cuda.mem_get_info()[0]) > left + (1 << 27):
        try:
            hogs.append(torch.empty(min(free - left, 32 << 30), dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:
            break
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
