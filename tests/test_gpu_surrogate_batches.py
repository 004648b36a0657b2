"""Training gradients of the surrogate at batch sizes around the kernels' edges, against the
FP64 network: one sample, a last workgroup or tile with few rows, more samples than
workgroups of the decoder's backward (several samples summed by one of them)."""
import numpy as np
import pytest

from oracle import surrogate as OS
from tests.helpers import rel_l2
from tests.test_gpu_surrogate import _decisive_params, _flat, _inputs, _unflat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 33, 255, 257, 520])
def test_surrogate_gradient_at_batch(lib, batch):
    import torch
    rw = lib
    coef, z, x = _inputs(torch, batch, 52)
    p = _decisive_params(51, x)
    sg = rw.Surrogate(max_batch=batch)
    sg.set_state(_flat(p))
    target = np.random.default_rng(53).normal(0, 0.3, (batch, 64, 64)).astype(np.float32)
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    sg.gradient(coef, z, torch.tensor(target, device="cuda"), loss=loss)
    torch.cuda.synchronize()
    ref_loss, ref_g = OS.loss_and_grads(p, x, target.astype(np.float64))
    g = _unflat(sg.get_state()["grads"], p)
    sg.close()
    assert abs(loss.item() - ref_loss) < 1e-5 * ref_loss
    for k in p:   # the bar of the gradient test: FP32 sums over the batch, 1e-4
        assert rel_l2(g[k], ref_g[k]) < 1e-4, (k, rel_l2(g[k], ref_g[k]))
