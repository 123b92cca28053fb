"""The BF16 products at the edges of their tiles: every output tile size, rows
that end inside a 16-byte vector, operands of fewer than 8 rows, K that ends
inside a stage, and the output layer's own kernel (a training step over two row
blocks, a rank below 64, a width that is no multiple of its tile)."""
import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (7, 5, 64), (8, 9, 128), (63, 65, 127), (130, 200, 129), (129, 2050, 65),
                                   (2049, 1500, 191),    # 128 x 128 tiles, ragged on every side
                                   (3900, 4007, 130),    # 256 x 256 tiles
                                   (4096, 3841, 64)])
def test_gemm_tile_edges(ta, tb, M, N, K):
    import torch
    from paper_2312_14832_amd import warmstart
    say(f"case gemm ta={ta} tb={tb} {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M + 31 * N + 7 * K)
    A = torch.randn((K, M) if ta else (M, K), generator=g).bfloat16()
    B = torch.randn((N, K) if tb else (K, N), generator=g).bfloat16()
    C = warmstart.gemm(A.cuda(), B.cuda(), ta, tb).cpu()
    A, B = (A.T if ta else A).float(), (B.T if tb else B).float()
    ref = A @ B
    # FP32 sums of K exact products, in any order: (K - 1) roundings of 2^-24
    # on partial sums below |A||B|, on both sides
    bound = 2 * K * 2.0 ** -24 * (A.abs() @ B.abs()) + 1e-30
    assert bool(((C - ref).abs() <= bound).all()), float(((C - ref).abs() / bound).max())


@pytest.mark.parametrize("rank,out_dim,B", [(64, 8200, 300), (40, 8193, 64), (64, 33, 257), (8, 8, 5), (72, 100, 20)])
def test_output_layer_step(rank, out_dim, B):
    """The BF16 training step's loss and output-layer gradients against FP64 of
    the same bfloat16 operands."""
    import torch
    from paper_2312_14832_amd import warmstart
    say(f"case output layer rank={rank} out={out_dim} B={B}")
    rng = np.random.default_rng(rank + out_dim + B)
    net = warmstart.Net(out_dim, in_dim=16, hidden=32, layers=1, rank=rank, max_batch=B, precision="bf16")
    p = net.init_params(3, out_bias=rng.standard_normal(out_dim))
    X = rng.standard_normal((B, 16)).astype(np.float32)
    Zs = rng.standard_normal((B, out_dim)).astype(np.float32)
    Xd, Zd = torch.from_numpy(X).cuda(), torch.from_numpy(Zs).cuda()
    Z = net.forward(Xd).cpu().numpy().astype(np.float64)
    loss = net.loss_grad(Xd, Zd)
    gb = net.grads()[-out_dim:].astype(np.float64)
    gW = net.grads()[-out_dim - rank * out_dim:-out_dim].astype(np.float64).reshape(rank, out_dim)
    d = Z - Zs
    # the step's predictions are the forward pass's, bit for bit, so the loss
    # differs by the summation order of FP64 and one FP32 rounding of each d
    assert abs(loss - np.mean(d * d)) <= 1e-6 * np.mean(d * d)
    dz = 2 * d / d.size
    # FP32 sums of B values, each with two roundings
    assert np.all(np.abs(gb - dz.sum(0)) <= (B + 3) * 2.0 ** -24 * np.abs(dz).sum(0) + 1e-30)

    def bf16(a):
        return torch.from_numpy(np.ascontiguousarray(a, np.float32)).bfloat16().double().numpy()

    W1, b1 = p[:16 * 32].reshape(16, 32), p[16 * 32:16 * 32 + 32]
    W2, b2 = p[544:544 + 32 * rank].reshape(32, rank), p[544 + 32 * rank:544 + 32 * rank + rank]
    h = bf16(np.maximum(bf16(X) @ bf16(W1) + b1, 0))
    a = bf16(h @ bf16(W2) + b2)
    ref = a.T @ bf16(dz)
    # an FP32 rounding ahead of bfloat16 can move an operand by one bfloat16
    # step (2^-8) here and there, on either side
    bound = 2.0 ** -7 * (np.abs(a).T @ np.abs(dz)) + 1e-30
    assert np.all(np.abs(gW - ref) <= bound), float((np.abs(gW - ref) / bound).max())
    net.close()
