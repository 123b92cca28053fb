"""lp_spmv_noalloc with in and out in the same memory: the product is that of
lp_spmv, bit for bit, in every layout."""
import numpy as np
import pytest

from paper_2312_14832_amd import gen
from gpu_helpers import say

pytestmark = pytest.mark.gpu


# a square K of 512- and 2048-entry row blocks; more rows than a launch's
# workgroups hold at once; several column slices
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,per_col,opt,slices", [(3000, 5, {}, 1), (3000, 5, dict(split_sums=1), 1),
                                                  (200000, 6, dict(slice_kib=4096), 1), (40000, 6, dict(slice_kib=64), 0)])
def test_product_in_place(lpmod, precision, n, per_col, opt, slices):
    import torch
    say(f"case spmv overlap {precision} {n} {opt}")
    data = gen.tiny_lp(3, n=n, m1=n // 3, m2=n - n // 3, per_col=per_col)
    p = lpmod.Problem(data, precision=precision, **opt)
    assert slices == 0 or p.layout() == (slices, slices)
    x = np.random.default_rng(1).standard_normal(n)
    for transpose in (False, True):
        want = p.spmv(x, transpose)
        # out is in; out begins inside in; out ends inside it
        for at_in, at_out in ((0, 0), (0, n // 2 + 1), (n // 2 + 1, 0)):
            buf = torch.zeros(2 * n, dtype=torch.float64, device="cuda")
            buf[at_in:at_in + n] = torch.from_numpy(x)
            torch.cuda.synchronize()
            p.spmv_noalloc(buf.data_ptr() + 8 * at_in, buf.data_ptr() + 8 * at_out, transpose)
            torch.cuda.synchronize()
            assert np.array_equal(buf[at_out:at_out + n].cpu().numpy(), want), (transpose, at_in, at_out)
