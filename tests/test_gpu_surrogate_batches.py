"""Training gradients of the surrogate at batch sizes around the kernels' edges, against the
FP64 network: one sample, a last workgroup or tile with few rows, more samples than
workgroups of the decoder's backward (several samples summed by one of them, more rows than the few-row products take) -- and
a captured forward after the weights have changed."""
import numpy as np
import pytest

from oracle import surrogate as OS
from tests.helpers import rel_l2
from tests.test_gpu_surrogate import _decisive_params, _flat, _inputs, _random_params, _unflat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 33, 255, 257, 512, 520])
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


@pytest.mark.parametrize("batch", [1, 40, 512, 513])
@pytest.mark.parametrize("precision,tol", [("SG_BF16X3", 1e-5), ("SG_BF16", 1e-2)])   # the bars of the forward test
def test_surrogate_forward_at_batch(lib, batch, precision, tol):
    import torch
    rw = lib
    coef, z, x = _inputs(torch, batch, 62)
    p = _random_params(61)
    sg = rw.Surrogate(max_batch=batch)
    sg.set_state(_flat(p))
    out = sg.forward(coef, z, precision=getattr(rw, precision))
    torch.cuda.synchronize()
    assert rel_l2(out.cpu().numpy(), OS.forward(p, x)[0]) < tol
    sg.close()


def test_captured_forward_sees_new_weights(lib):
    import torch
    rw = lib
    coef, z, _ = _inputs(torch, 48, 72)
    target = torch.randn(48, 64, 64, device="cuda", generator=torch.Generator("cuda").manual_seed(73))
    sg = rw.Surrogate(max_batch=48)
    sg.set_state(_flat(_random_params(71)))
    out = torch.zeros(48, 64, 64, device="cuda")
    sg.forward(coef, z, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sg.forward(coef, z, out=out)
    for step in range(4):
        if step == 2:
            sg.set_state(_flat(_random_params(74)))
        else:
            sg.gradient(coef, z, target)
            sg.adam(1e-3)
        eager = sg.forward(coef, z).clone()
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), step
    sg.close()
