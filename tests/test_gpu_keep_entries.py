"""The two ways the products' entries are read, on either side of the size at
which one takes over from the other: products equal to the oracle's."""
import numpy as np
import pytest

from paper_2312_14832_amd import gen
from gpu_helpers import say

pytestmark = pytest.mark.gpu


# bytes of both matrices' entries and 9 n + 7 m values, against 256 MiB:
# just below and just above it, one slice and several
@pytest.mark.parametrize("precision,n,m1,m2,per_col", [("fp64", 400000, 90000, 110000, 23), ("fp64", 400000, 90000, 110001, 24),
                                                      ("mixed", 500000, 100000, 90000, 29),
                                                      ("mixed", 500000, 100000, 90001, 31)])
def test_products_on_either_side(lpmod, oracle_mod, precision, n, m1, m2, per_col):
    say(f"case keep entries {precision} {n} {per_col}")
    p = gen.tiny_lp(5, n=n, m1=m1, m2=m2, per_col=per_col)
    h = lpmod.Problem(p, precision=precision)
    o = oracle_mod.Oracle(p)
    rng = np.random.default_rng(3)
    # rows of up to some 100 entries: (100 + 3) u of a sum of magnitudes that is
    # at most 5 times the normal result's norm, and 4e-13 for the scaling factors
    tol = 512 * (2.0 ** -53 if precision == "fp64" else 2.0 ** -24) + 4e-13
    for transpose, size in ((False, p.n), (True, p.m)):
        x = rng.standard_normal(size).astype(np.float32).astype(np.float64)
        got, want = h.spmv(x, transpose=transpose), o.spmv(x, transpose=transpose)
        assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want), transpose
