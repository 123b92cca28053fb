"""Reading a batch's results in order (fetched several at a time), out of order
and in part gives the same points, also after another solve."""
import numpy as np
import pytest

from paper_2312_14832_amd import gen
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
# the second: instances whose points do not fit one fetch together
@pytest.mark.parametrize("sizes", [[3, 255, 256, 257, 40, 300, 17, 1000, 9], [90000, 700, 120000, 800, 100000, 600]])
def test_results_in_any_order(lpmod, sizes, precision):
    say(f"case batch results {sizes} {precision}")
    lps = [gen.tiny_lp(i, n=n, m1=max(n // 5, 1), m2=max(n // 4, 2), per_col=min(3, max(n // 5, 1))) for i, n in enumerate(sizes)]
    b = lpmod.Batch(lps, precision=precision)
    for steps in (10, 30):
        b.solve(1e-30, steps)
        order = [b.result(i) for i in range(len(lps))]
        again = [b.result(i) for i in range(len(lps))]
        back = [b.result(i) for i in reversed(range(len(lps)))][::-1]
        for i, p in enumerate(lps):
            assert order[i][0].shape == (p.n,) and order[i][1].shape == (p.m,)
            for a, c, d in zip(order[i][:3], again[i][:3], back[i][:3]):
                assert np.array_equal(a, c) and np.array_equal(a, d)
            assert order[i][3] == back[i][3] and order[i][3]["iterations"] == steps
            alone = lpmod.Problem(p, precision=precision)
            alone.solve(1e-30, steps)
            x, y, _, _ = alone.result()
            # the same steps in another summation order, ten or thirty of them
            tol = 1e-11 if precision == "fp64" else 2e-3
            for u, v in ((order[i][0], x), (order[i][1], y)):
                assert np.linalg.norm(u - v) <= tol * (1 + np.linalg.norm(v))
    b.close()
