"""Reading parts of a batch's points (x, y or lambda alone, now one and now the
other) in order and out of it gives what reading all of them does."""
import ctypes as C

import numpy as np
import pytest

from paper_2312_14832_amd import gen
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes", [[3, 255, 256, 257, 40, 300, 17, 1000, 9, 20], [90000, 700, 120000, 800, 100000, 600]])
def test_parts_of_results(lpmod, sizes, precision):
    say(f"case batch result parts {sizes} {precision}")
    lps = [gen.tiny_lp(i, n=n, m1=max(n // 5, 1), m2=max(n // 4, 2), per_col=min(3, max(n // 5, 1))) for i, n in enumerate(sizes)]
    b = lpmod.Batch(lps, precision=precision)
    b.solve(1e-30, 20)
    want = [b.result(i)[:3] for i in reversed(range(len(lps)))][::-1]

    def part(i, which):
        out = [np.full(p, np.nan) if k in which else None for k, p in zip("xyl", (lps[i].n, lps[i].m, lps[i].n))]
        ptr = [None if a is None else a.ctypes.data_as(C.POINTER(C.c_double)) for a in out]
        assert lpmod.library().lp_batch_result(b.h, i, *ptr, None) == 0
        for a, w in zip(out, want[i]):
            assert a is None or np.array_equal(a, w), (i, which)

    every = range(len(lps))
    for reads in ([(i, "x") for i in every], [(i, w) for i in every for w in "xyl"], [(i, w) for w in ("y", "xl") for i in every],
                  [(i, ("x", "yl", "xyl", "l")[i % 4]) for i in every] + [(i, "xyl") for i in every],
                  [(i, "xyl") for i in every if i != 4] + [(4, "y"), (5, "x"), (5, "y"), (4, "l")]):
        b.solve(1e-30, 7)   # drops what was fetched
        b.solve(1e-30, 20)
        for i, which in reads:
            part(i, which)
    b.close()
