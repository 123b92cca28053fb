"""The slot in two kernels (LPs of one column slice): its block sizes, row
forms, check groups and window lengths, against the oracle's own steps."""
import numpy as np
import pytest

from paper_2312_14832_amd import gen
from gpu_helpers import say

pytestmark = pytest.mark.gpu


def uneven_lp(seed, n, m1, m2, longest):
    """Short columns with some long ones: rows of K' that keep a wavefront or a
    whole workgroup each, and empty ones."""
    rng = np.random.Generator(np.random.PCG64(seed))
    counts = rng.choice([0, 1, 2, 3, 5, 9, 65, 130], size=n, p=[.1, .25, .25, .2, .1, .05, .03, .02]).astype(np.int64)
    counts[:3] = longest
    return gen.certificate_lp(rng, m1, m2, counts)


CASES = [
    # columns and rows at a block's edge, a window of odd length (the controller ends in its second copy)
    ("tiny 256", lambda: gen.tiny_lp(1, n=256, m1=100, m2=156), dict(window=7)),
    ("tiny 257", lambda: gen.tiny_lp(2, n=257, m1=1, m2=512), dict(window=1, check_every=10)),
    ("tiny 513", lambda: gen.tiny_lp(3, n=513, m1=200, m2=57), dict(check_every=7, use_graph=0)),
    ("uneven", lambda: uneven_lp(4, 3000, 700, 800, 900), dict()),
    ("uneven split", lambda: uneven_lp(5, 3000, 700, 800, 600), dict(split_sums=1, check_every=6)),
    # 512, 1024 and 2048 nonzeros to a block
    ("medium 512", lambda: gen.tiny_lp(6, n=40000, m1=8000, m2=12000, per_col=6), dict(check_every=24)),
    ("medium 1024", lambda: gen.tiny_lp(7, n=60000, m1=10000, m2=15001, per_col=8), dict(window=33)),
    ("medium 2048", lambda: gen.tiny_lp(8, n=100000, m1=20000, m2=30000, per_col=7), dict(check_every=16)),
    # more row blocks than workgroups
    ("blocks past the grid", lambda: gen.tiny_lp(9, n=260000, m1=30000, m2=70000, per_col=9), dict(check_every=16)),
]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name,make,opt", CASES, ids=[c[0] for c in CASES])
def test_fused_slot_matches_oracle(lpmod, oracle_mod, name, make, opt, precision):
    say(f"case fused slot {name} {precision}")
    data = make()
    # FP32: 8 steps, each within the single step's 64 u normwise and growing
    # by less than a factor of two a step; FP64: inside the first checks'
    # horizon, where the method's own sensitivity stays far below 1e-10
    steps, tol = (48, 1e-10) if precision == "fp64" else (8, 256 * 64 * 2.0 ** -24)
    p = lpmod.Problem(data, precision=precision, persistent=0, **opt)
    assert p.layout() == (1, 1)
    p.solve(1e-30, steps)
    s = lpmod.unpack_state(p.get_state(), data.n, data.m)
    o = oracle_mod.Oracle(data, check_every=opt.get("check_every", 64))
    o.solve(1e-30, steps)
    t = o.get_state()
    for k in ("k", "t", "attempts", "restarts"):
        assert s[k] == t[k], (k, s[k], t[k])
    for k in ("x", "y", "Kx", "KTy", "xbar", "ybar", "Kxbar", "KTybar", "x0", "y0"):
        err = np.linalg.norm(s[k] - t[k]) / max(np.linalg.norm(t[k]), 1e-300)
        assert err < tol, (k, err)
    # the same again, resumed in the middle, bit for bit
    q = lpmod.Problem(data, precision=precision, persistent=0, **opt)
    half = steps // 2 // opt.get("check_every", 64) * opt.get("check_every", 64) or steps // 2
    if half % opt.get("check_every", 64) == 0:
        q.solve(1e-30, half)
        q.set_state(q.get_state())
        q.solve(1e-30, steps)
        assert np.array_equal(q.get_state(), p.get_state())
