"""FP32 gradients of a training step, contracted in parts and finished in place,
against FP64."""
import pytest
import torch

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,hidden,rank,out_dim", [(64, 64, 64, 30001), (200, 130, 96, 5003), (1000, 48, 8, 2000)])
def test_fp32_step_in_parts(B, hidden, rank, out_dim):
    """Loss and every gradient against FP64, where dL/dalpha is summed in parts
    over out_dim and the step's epilogue works in place on one part."""
    from paper_2312_14832_amd import warmstart
    say(f"case fp32 step in parts {B} {hidden} {rank} {out_dim}")
    net = warmstart.Net(out_dim, in_dim=24, hidden=hidden, layers=2, rank=rank, max_batch=B, precision="fp32")
    p = torch.from_numpy(net.init_params(2)).double().cuda()
    g = torch.Generator(device="cuda").manual_seed(B)
    X, Z = torch.randn(B, 24, generator=g, device="cuda"), torch.randn(B, out_dim, generator=g, device="cuda")
    loss = net.loss_grad(X, Z)
    got = torch.from_numpy(net.grads()).double().cuda()
    dims, at, layers = [24, hidden, hidden, rank, out_dim], 0, []
    for a, b in zip(dims[:-1], dims[1:]):
        layers.append((p[at:at + a * b].reshape(a, b), p[at + a * b:at + a * b + b]))
        at += a * b + b
    acts = [X.double()]
    for i, (w, c) in enumerate(layers):
        h = acts[-1] @ w + c
        acts.append(h.clamp(min=0) if i < 2 else h)
    d = acts[-1] - Z.double()
    want = float((d * d).mean())
    assert abs(loss - want) <= 1e-5 * want
    dy, grads = 2 * d / d.numel(), []
    for i in reversed(range(len(layers))):
        if i < 2:
            dy = dy * (acts[i + 1] > 0)
        grads = [acts[i].t().contiguous() @ dy, dy.sum(0)] + grads
        dy = dy @ layers[i][0].t().contiguous()
    at = 0
    for ref in grads:
        part = got[at:at + ref.numel()].reshape(ref.shape)
        at += ref.numel()
        # chains of at most out_dim + some roundings whose errors are random:
        # 8 sqrt(out_dim) units normwise, and a ReLU's sign that rounding moves
        assert float((part - ref).norm()) <= 8 * out_dim ** 0.5 * 2.0 ** -24 * float(ref.norm()) + 1e-30, ref.shape
    net.close()
