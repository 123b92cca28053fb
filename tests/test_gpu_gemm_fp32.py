"""FP32 matrix products at the edges of their tiles, vectors and stages, in both
tile sizes, against the product in FP64."""
import pytest
import torch

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (3, 66, 2), (64, 64, 16), (65, 63, 17), (130, 127, 47), (61, 129, 300),
                                   # 128-wide tiles: whole ones, and ragged in every direction
                                   (4096, 4096, 16), (4033, 4099, 37)])
def test_fp32_gemm_edges(lpmod, M, N, K, ta, tb):
    from paper_2312_14832_amd import warmstart
    say(f"case fp32 gemm {M} {N} {K} {ta} {tb}")
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N + K)
    A = torch.randn((K, M) if ta else (M, K), device="cuda", generator=g)
    B = torch.randn((N, K) if tb else (K, N), device="cuda", generator=g)
    C = warmstart.gemm(A, B, bool(ta), bool(tb), precision="fp32").double()
    a, b = (A.t() if ta else A).double().contiguous(), (B.t() if tb else B).double().contiguous()
    # a chain of K fused multiply-adds: at most K roundings of partial sums of the magnitudes
    bound = 1.01 * K * 2.0 ** -24 * (a.abs() @ b.abs())
    assert bool(((C - a @ b).abs() <= bound).all())
