"""A stack of a call does not depend on the others: not on a neighbour with coefficients at the end of
the range (whose own phase is then not finite), nor on how many terms the neighbours have."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["FORM_FOURIER", "FORM_CHIRPZ"])
@pytest.mark.parametrize("terms", [0, 1, 5, 23, 24, 25, 36])
def test_neighbours_at_the_end_of_the_range(lib, form, terms):
    import torch
    rw = lib
    w = W.fourier_plain(n_stacks=1, seed=3)
    plan = rw.Plan(form=getattr(rw, form), **w["optics"], nx=16, ny=16, dx=30.0, dy=30.0, z=[-50.0, 80.0],
                   e_inc=w["e_inc"], n_pupil=48)
    rng = np.random.default_rng(terms)
    st = [dict(x0=5.0 * b, z_offset=9.0 * b, zernike=rng.normal(0, 0.05, terms)) for b in range(3)]
    alone = [plan.compute([s]) for s in st]
    call = [st[0], dict(zernike=np.full(max(terms, 1), 1e308)), st[1], dict(zernike=np.full(max(terms, 1), -1e308)), st[2]]
    E, I = plan.compute(call)
    torch.cuda.synchronize()
    plan.close()
    for b, (e, i) in zip((0, 2, 4), alone):
        assert torch.equal(E[b], e[0]) and torch.equal(I[b], i[0])
