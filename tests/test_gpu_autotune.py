"""Handles whose layout is chosen by timing (autotune=1): products and steps
against the oracle, and the products of lp_spmv and of the solve the same."""
import numpy as np
import pytest

from paper_2312_14832_amd import gen
from gpu_helpers import ints_equal, say, vec_diff

pytestmark = pytest.mark.gpu


def uneven_lp(seed, n, m):
    """Short columns and one in thirty of 65 to 200 entries: rows of K' that split sums keep among the short ones."""
    rng = np.random.Generator(np.random.PCG64(seed))
    counts = np.where(rng.random(n) < 1 / 30, rng.integers(65, 201, n), rng.integers(1, 9, n))
    return gen.certificate_lp(rng, m // 2, m - m // 2, counts)


CASES = [
    # one slice by default: a slot of two kernels unless slices win by whole slots
    ("small", lambda: gen.tiny_lp(0), dict(), "fp64"),
    ("medium", lambda: gen.tiny_lp(2, n=23457, m1=4401, m2=6602, per_col=6), dict(), "fp64"),
    ("uneven", lambda: uneven_lp(3, 60000, 30000), dict(), "fp64"),
    ("uneven split", lambda: uneven_lp(3, 60000, 30000), dict(split_sums=1), "mixed"),
    ("one slice, many blocks", lambda: uneven_lp(4, 250000, 100000), dict(), "mixed"),
    # several slices by default, with one as good
    ("slices", lambda: gen.tiny_lp(5, n=40000, m1=8000, m2=12000, per_col=6), dict(slice_kib=64), "fp64"),
    ("slices split", lambda: gen.tiny_lp(5, n=40000, m1=8000, m2=12000, per_col=6), dict(slice_kib=64, split_sums=1), "fp64"),
    ("K alone in slices", lambda: gen.tiny_lp(6, n=400000, m1=60000, m2=60000, per_col=5), dict(), "fp64"),
    # entries past the last-level cache
    ("large", lambda: gen.tiny_lp(7, n=420000, m1=90000, m2=110000, per_col=25), dict(slice_kib=4096), "fp64"),
    ("dense row", lambda: gen.pagerank_lp(1, 100000), dict(), "fp64"),
]


@pytest.mark.parametrize("name,make,opt,precision", CASES, ids=[c[0] for c in CASES])
def test_tuned_handle(lpmod, oracle_mod, name, make, opt, precision):
    say(f"case autotune {name}")
    data = make()
    p = lpmod.Problem(data, precision=precision, autotune=1, persistent=0, **opt)
    say("  layout", p.layout_blocks(0), p.layout_split(0), p.layout_blocks(1), p.layout_split(1))
    o = oracle_mod.Oracle(data)
    rng = np.random.default_rng(1)
    unit = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    for transpose, size in ((False, data.n), (True, data.m)):
        x = rng.standard_normal(size).astype(np.float32).astype(np.float64)
        want = o.spmv(x, transpose=transpose)
        # rows of up to some 200 short sums: 256 units of a sum of magnitudes that
        # is at most 5 times the normal result's norm, and the scaling's 4e-13
        assert np.linalg.norm(p.spmv(x, transpose=transpose) - want) <= (1280 * unit + 4e-13) * np.linalg.norm(want)
    steps = 24 if precision == "fp64" else 1
    p.solve(1e-30, steps)
    o.solve(1e-30, steps)
    sg, so = lpmod.unpack_state(p.get_state(), data.n, data.m), o.get_state()
    assert ints_equal(sg, so)
    worst, where = vec_diff(sg, so)
    # FP64: far inside the steps over which the method keeps rounding below
    # 1e-10; FP32: one step, 64 units normwise
    assert worst < (1e-10 if precision == "fp64" else 64 * unit), (where, worst)
    # the solve's products are those of lp_spmv, bit for bit
    assert np.array_equal(p.spmv(sg["x"]), sg["Kx"])
    assert np.array_equal(p.spmv(sg["y"], transpose=True), sg["KTy"])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("rows", [0, 5])
def test_nothing_to_tune(lpmod, rows, precision):
    """No rows, or rows without entries."""
    say(f"case autotune without entries {rows} {precision}")
    n = 40
    data = gen.LPData(rows, n, 0, np.zeros(rows + 1, np.int32), np.zeros(0, np.int32), np.zeros(0),
                      np.linspace(-1, 1, n), -np.ones(rows), np.zeros(n), np.full(n, 3.0))
    for opt in (dict(), dict(persistent=0)):
        p = lpmod.Problem(data, precision=precision, autotune=1, **opt)
        info = p.solve(1e-6, 1000)
        assert info["status"] == "OPTIMAL"
        assert np.allclose(p.result()[0], np.where(data.c > 0, 0.0, 3.0), atol=1e-4)
        assert np.array_equal(p.spmv(np.ones(n)), np.zeros(rows))
