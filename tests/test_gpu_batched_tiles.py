"""Tile classes and the fold of the batched emitters against the FP64 oracle: every pupil size on
the 32- and the 64-row tiles at crops on and beside their edges, and emitter counts that leave the
last group of the fold short."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_fourier_stack, oracle_optics, rel_l2

pytestmark = pytest.mark.gpu
TOL = 1e-5   # the bar of the FP32 forms


# emitters: 5 leaves one emitter a group, 1700 some (1024 workgroups of 256 cells on 256 CUs), the
# last group not full
@pytest.mark.parametrize("n_pupil", [32, 64, 96, 128])
@pytest.mark.parametrize("n", [5, 1700])
@pytest.mark.parametrize("crops", [(1, 16, 31, 32), (33, 47, 63, 64), (32, 33, 2, 64)])
def test_batched_tile_classes(lib, n_pupil, n, crops):
    import torch
    rw = lib
    w = W.batched(n_emitters=n, seed=41)
    o = w["optics"]
    S = np.array(crops)[np.arange(n) % 4]
    D = 1 + np.arange(n) % 3 if n < 10 else np.ones(n, dtype=int)
    em = rw.make_emitters(w["x0"], w["y0"], w["z_e"], S, D, w["zernike"])
    off = rw.batch_offsets(em)
    b = rw.Batch(na=o["na"], wavelength=o["wavelength"], n_i=o["n_i"], pixel=w["dx"], plane_pitch=w["dz"],
                 max_emitters=n, n_pupil=n_pupil, e_inc=w["e_inc"])
    I = torch.full((int(off[-1]),), -1.0, device="cuda")
    E = torch.zeros(3 * int(off[-1]), dtype=torch.complex64, device="cuda")
    b.compute(em, I=I, E=E)
    torch.cuda.synchronize()
    b.close()
    opt = oracle_optics(w, gl=False)
    assert (I >= 0).all()
    for i in (0, 1, 2, 3, 4, n // 2, n - 4, n - 3, n - 2, n - 1):
        z = (np.arange(D[i]) - 0.5 * (D[i] - 1)) * w["dz"] - w["z_e"][i]
        ref = oracle_fourier_stack(opt, n_pupil, S[i], S[i], w["dx"], w["dx"], z, zernike=w["zernike"][i],
                                   x0=w["x0"][i], y0=w["y0"][i])
        e = E[3 * off[i]:3 * off[i + 1]].view(D[i], 3, S[i], S[i]).cpu().numpy()
        v = I[off[i]:off[i + 1]].view(D[i], S[i], S[i]).cpu().numpy()
        assert rel_l2(e, ref) < TOL, (i, S[i])
        assert rel_l2(v, (np.abs(ref) ** 2).sum(axis=1)) < TOL, (i, S[i])
