"""Shared-matrix batches of at most four members (one group, walked plainly) and
of groups in which some workgroups have nothing: members that end at different
steps, each meeting its tolerance and unmoved by what the others still do."""
import numpy as np
import pytest

from paper_2312_14832_amd import gen
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("count,n", [(1, 600), (2, 257), (3, 600), (4, 1000), (35, 300)])
def test_members_end_apart(lpmod, oracle_mod, count, n, precision):
    say(f"case shared narrow {count} {n} {precision}")
    base = gen.parametric_base(4, n=n, m1=n // 4, m2=n // 4)
    lps = [gen.parametric_instance(base, s) for s in range(count)]
    sh = lpmod.Shared(lps, precision=precision, window=16)
    sh.solve(1e-4, 100000)
    ends = [sh.info(i)["iterations"] for i in range(count)]
    assert count < 3 or len(set(ends)) > 1
    first = int(np.argmin(ends))
    for i in sorted({0, first, count - 1}):
        assert sh.info(i)["status"] == "OPTIMAL"
        x, y = sh.result(i)[:2]
        assert oracle_mod.Oracle(lps[i]).eval_unscaled(x, y)["rel_kkt"] <= 1e-4 * (1 + 1e-6)
    # the first to end, stopped there: the same point, bit for bit
    again = lpmod.Shared(lps, precision=precision, window=16)
    again.solve(1e-4, ends[first])
    for a, b in zip(sh.result(first)[:3], again.result(first)[:3]):
        assert np.array_equal(a, b)
