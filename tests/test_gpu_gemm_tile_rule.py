"""BF16 products at shapes where the rule picks each output tile, ragged in every
direction."""
import pytest
import torch

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("M,N,K", [(1003, 1001, 777),     # 64 x 64 tiles
                                   (2049, 3001, 777),     # 128 x 128
                                   (3001, 2999, 1500)])   # 256 x 256
def test_gemm_at_each_tile(ta, tb, M, N, K):
    from paper_2312_14832_amd import warmstart
    say(f"case gemm tile rule ta={ta} tb={tb} {M}x{N}x{K}")
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((K, M) if ta else (M, K), generator=g, device="cuda").bfloat16()
    B = torch.randn((N, K) if tb else (K, N), generator=g, device="cuda").bfloat16()
    C = warmstart.gemm(A, B, ta, tb).double()
    a, b = (A.t() if ta else A).double().contiguous(), (B.t() if tb else B).double().contiguous()
    # FP32 sums of K exact products, in any order
    assert bool(((C - a @ b).abs() <= K * 2.0 ** -24 * (a.abs() @ b.abs()) + 1e-30).all())
