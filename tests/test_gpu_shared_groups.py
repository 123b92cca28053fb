"""Shared-matrix batches at the edges of the instance groups (a padded last
group, one group alone, more groups than XCDs, FP32's two widths) and of the
entries that a row's lanes hold at a time, against each member's oracle."""
import numpy as np
import pytest

from paper_2312_14832_amd import gen
from gpu_helpers import say

pytestmark = pytest.mark.gpu


def uneven_family(count, n, m1, m2, seed=3):
    """One K with empty, short and long rows both ways, each member its own c and q."""
    rng = np.random.Generator(np.random.PCG64(seed))
    counts = rng.choice([0, 1, 4, 5, 8, 15, 16, 17, 33], size=n).astype(np.int64)
    counts = np.minimum(counts, m1 + m2)
    base = gen.certificate_lp(rng, m1, m2, counts)
    out = []
    for _ in range(count):
        c = base.c + 0.3 * rng.standard_normal(n)
        q = base.q + 0.3 * rng.standard_normal(m1 + m2)
        out.append(gen.LPData(m=base.m, n=base.n, m1=m1, row_ptr=base.row_ptr, col=base.col, val=base.val, c=c, q=q,
                              l=base.l, u=base.u))
    return out


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("count,n,m1,m2", [(2, 401, 100, 57), (8, 257, 1, 70), (9, 301, 60, 0), (17, 700, 0, 301),
                                           (33, 130, 20, 30), (64, 90, 11, 23), (145, 65, 9, 13)])
def test_shared_groups_match_oracle(lpmod, oracle_mod, count, n, m1, m2, precision):
    say(f"case shared groups {count} {n} {m1} {m2} {precision}")
    lps = uneven_family(count, n, m1, m2)
    # 8 steps: FP32 each within the single step's 64 u normwise and growing by
    # less than a factor of two a step; FP64 the per-step bound of the lockstep
    # tests (an input moved by one rounding moves the oracle's own 8 steps by at
    # most 1e-14 here; by 48 steps it moves one member of the 17 by 5e-9)
    steps, tol = 8, 1e-10 if precision == "fp64" else 256 * 64 * 2.0 ** -24
    sh = lpmod.Shared(lps, precision=precision)
    rng = np.random.default_rng(7)
    starts = {i: (rng.standard_normal(n), rng.standard_normal(m1 + m2)) for i in {0, count - 1}}
    for i, (x0, y0) in starts.items():
        sh.set_start(i, x0, y0, 0.0)
    sh.solve(1e-30, steps)
    some = sorted({0, 1, count // 2, count - 2, count - 1})
    for i in some:
        o = oracle_mod.Oracle(lps[i])
        if i in starts:
            o.set_start(*starts[i])
        o.solve(1e-30, steps)
        s, t = lpmod.unpack_state(sh.get_state(i), n, m1 + m2), o.get_state()
        for k in ("k", "t", "attempts", "restarts"):
            assert s[k] == t[k], (i, k, s[k], t[k])
        for k in ("x", "y", "Kx", "KTy", "xbar", "ybar", "Kxbar", "KTybar", "x0", "y0"):
            err = np.linalg.norm(s[k] - t[k]) / max(np.linalg.norm(t[k]), 1e-300)
            assert err < tol, (i, k, err)
    # the states into another handle and on, the same as going on here
    other = lpmod.Shared(lps, precision=precision)
    for i in range(count):
        other.set_state(i, sh.get_state(i))
    for i in range(count):
        sh.set_state(i, other.get_state(i))
    sh.solve(1e-30, steps + 4)
    other.solve(1e-30, steps + 4)
    for i in some:
        assert np.array_equal(sh.get_state(i), other.get_state(i)), i
