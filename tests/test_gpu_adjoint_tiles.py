"""The adjoint's tiles against the FP64 gradient oracle: pupils of less and of more than one
workgroup's 256 rows, planes of less and of more than a 64 x 64 chunk along either axis, calls of
more stacks than one launch takes, and gradients that need the operand scales."""
import numpy as np
import pytest

import workloads as W
from oracle import adjoint as OA
from oracle import fourier as OF
from tests.helpers import oracle_optics, rel_l2

pytestmark = pytest.mark.gpu
TOL = 1e-5   # the bar of the FP32 forms


def _run(rw, n_pupil, nx, ny, nz, n_stacks, gradient):
    """Gradients here and from the oracle for dL/dI = gradient(I) of the oracle's intensities."""
    import torch
    w = W.adjoint(n_stacks=n_stacks, n_pupil=n_pupil, nx=16, nz=nz, seed_truth=11)
    rng = np.random.default_rng(n_pupil + nx)
    shifts = [(rng.uniform(-50, 50), rng.uniform(-50, 50), rng.uniform(-200, 200)) for _ in range(n_stacks)]
    opt, o = oracle_optics(w, gl=False), w["optics"]
    geom = OF.pupil_geometry(n_pupil, opt)
    w0 = w["w0_eval"].astype(np.float32)
    E, I = OA.forward(geom, opt, w["c_eval"], w0.astype(np.float64), shifts, nx, ny, w["dx"], w["dy"], w["z"])
    g = gradient(I).astype(np.float32)
    plan = rw.Plan(form=rw.FORM_FOURIER, na=o["na"], wavelength=o["wavelength"], n_i=o["n_i"], nx=nx, ny=ny, dx=w["dx"],
                   dy=w["dy"], z=w["z"], e_inc=w["e_inc"], n_pupil=n_pupil)
    m = torch.tensor(w0, device="cuda")
    st = [dict(x0=x, y0=y, z_offset=z, zernike=w["c_eval"], phase_map=m) for x, y, z in shifts]
    Et = torch.tensor(E.astype(np.complex64), device="cuda")

    def here(scale=1.0):
        dc, dw = plan.adjoint(st, Et, torch.tensor(g, device="cuda") * scale, 21)
        torch.cuda.synchronize()
        return dc.double().cpu().numpy(), dw.double().cpu().numpy()

    ref = OA.gradient(geom, opt, w["c_eval"], w0.astype(np.float64), shifts, nx, ny, w["dx"], w["dy"], w["z"],
                      g.astype(np.float64))
    return here, ref


@pytest.mark.parametrize("n_pupil,nx,ny,nz,n_stacks", [
    (33, 16, 16, 1, 1), (300, 64, 16, 2, 1), (257, 16, 80, 2, 1), (64, 80, 144, 3, 2), (130, 144, 64, 5, 2),
    (32, 16, 16, 2, 67)])
def test_adjoint_tiles(lib, n_pupil, nx, ny, nz, n_stacks):
    here, (dc_ref, dw_ref) = _run(lib, n_pupil, nx, ny, nz, n_stacks, lambda I: I - 0.3 * I.max())
    dc, dw = here()
    assert rel_l2(dc, dc_ref) < TOL
    assert rel_l2(dw, dw_ref) < TOL


def test_adjoint_of_planes_of_unequal_scale(lib):
    """A plane without gradient, one 1e-12 of the others and one whose gradient sits on the
    darkest pixels; the result is exactly linear in powers of two of dL/dI."""
    def gradient(I):
        g = I - 0.3 * I.max()
        g[0, 0] = 0.0
        g[0, 1] *= 1e-12
        g[1, 2] = np.where(I[1, 2] < np.quantile(I[1, 2], 0.1), 1.0 / (I[1, 2] + 1e-3 * I.min()), 0.0)
        g[1, 2] *= np.abs(g[0, 2]).max() / g[1, 2].max()
        return g

    here, (dc_ref, dw_ref) = _run(lib, 48, 32, 48, 4, 2, gradient)
    dc, dw = here()
    assert rel_l2(dc, dc_ref) < TOL
    assert rel_l2(dw, dw_ref) < TOL
    for e in (-40, 30):
        dc2, dw2 = here(2.0 ** e)
        assert np.array_equal(dc2, dc * 2.0 ** e) and np.array_equal(dw2, dw * 2.0 ** e)
