"""How solves in the two-kernel slot end and go on: an optimum, an infeasible
LP, a re-check in FP64 that fails and lets the loop go on (mixed precision), the
iteration limit and a resume, in slots of either parity, windows of any length
and with check kernels every few slots."""
import numpy as np
import pytest

from paper_2312_14832_amd import gen
from lp_helpers import farkas_ratios
from gpu_helpers import say

pytestmark = pytest.mark.gpu

# what a window holds and how it is launched changes no bit of a solve: slots
# after a check that fell due, or after the end, do nothing until the host looks
WINDOWS = [dict(window=64), dict(window=7), dict(window=1), dict(window=33, use_graph=0)]


def ends(lpmod, data, tol, iters, **opt):
    """(info, point and state) of the same solve at each of WINDOWS."""
    out = []
    for w in WINDOWS:
        p = lpmod.Problem(data, persistent=0, **opt, **w)
        assert p.layout() == (1, 1)
        info = p.solve(tol, iters)
        x, y, lam, _ = p.result()
        out.append((info, (x, y, lam, p.get_state())))
        p.close()
    for info, arrays in out[1:]:
        for k in ("status", "iterations", "attempts", "restarts", "omega", "eta", "pobj", "rel_kkt"):
            assert info[k] == out[0][0][k], (k, info[k], out[0][0][k])
        for a, b in zip(arrays, out[0][1]):
            assert np.array_equal(a, b)
    return out[0]


@pytest.mark.parametrize("check_every", [10, 64, 7])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("seed", [0, 2])
def test_optimum(lpmod, oracle_mod, seed, precision, check_every):
    say(f"case fused optimum {seed} {precision} check_every={check_every}")
    data = gen.tiny_lp(seed)
    info, (x, y, _, _) = ends(lpmod, data, 1e-4, 200000, precision=precision, check_every=check_every)
    assert info["status"] == "OPTIMAL" and info["iterations"] % check_every == 0
    assert oracle_mod.Oracle(data).eval_unscaled(x, y)["rel_kkt"] <= 1e-4 * (1 + 1e-6)


@pytest.mark.parametrize("tol", [1e-5, 1e-6, 2e-7])
def test_failed_recheck_goes_on(lpmod, oracle_mod, tol):
    """Tolerances down to what FP32 products can tell, where the FP64 re-check of
    a passed test can fail."""
    say(f"case fused re-check {tol}")
    data = gen.tiny_lp(1)
    info, (x, y, _, _) = ends(lpmod, data, tol, 20000, precision="mixed", check_every=24)
    ev = oracle_mod.Oracle(data).eval_unscaled(x, y)
    if info["status"] == "OPTIMAL":
        assert ev["rel_kkt"] <= tol * (1 + 1e-6), ev
    else:
        assert info["status"] == "ITERATION_LIMIT" and info["iterations"] == 20000


@pytest.mark.parametrize("kind,status", [("primal", "PRIMAL_INFEASIBLE"), ("dual", "DUAL_INFEASIBLE")])
def test_infeasible(lpmod, kind, status):
    say(f"case fused infeasible {kind}")
    data = gen.infeasible_lp(0, kind)
    info, (x, y, _, _) = ends(lpmod, data, 1e-8, 600000)
    assert info["status"] == status
    dobj, dres, pobj, pres = farkas_ratios(data, x, y)
    if kind == "primal":
        assert dobj > 0 and dres <= 1e-8 * dobj * (1 + 1e-6)
    else:
        assert pobj < 0 and pres <= 1e-8 * -pobj * (1 + 1e-6)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,check_every,window", [(1000, 4, 7), (1000, 6, 64), (60000, 4, 5)])
def test_resume_at_a_check(lpmod, precision, n, check_every, window):
    """Stopped at a check, saved and resumed: the same bits as in one go."""
    say(f"case fused resume {precision} {n} {check_every} {window}")
    data = gen.tiny_lp(4, n=n, m1=n // 5, m2=n // 4 + 1)
    opt = dict(precision=precision, persistent=0, check_every=check_every, window=window)
    p, q = lpmod.Problem(data, **opt), lpmod.Problem(data, **opt)
    assert p.layout() == (1, 1)
    p.solve(1e-30, 5 * check_every)
    q.solve(1e-30, 3 * check_every)
    q.set_state(q.get_state())
    q.solve(1e-30, 5 * check_every)
    assert np.array_equal(p.get_state(), q.get_state())


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_time_limit_and_on(lpmod, oracle_mod, precision):
    """The time limit's point is the one it reports on, and the saved state
    goes on to an optimum."""
    say(f"case fused time limit {precision}")
    data = gen.tiny_lp(0)
    o = oracle_mod.Oracle(data)
    p = lpmod.Problem(data, precision=precision, persistent=0, window=7)
    info = p.solve(1e-30, 10 ** 9, 0.05)
    assert info["status"] == "TIME_LIMIT" and info["iterations"] > 0
    x, y, _, _ = p.result()
    ev = o.eval_unscaled(x, y)
    # the reported quantities come from products kept through the averages: far
    # from the optimum's last digits in either precision
    assert info["pobj"] == pytest.approx(ev["pobj"], rel=1e-3 if precision == "mixed" else 1e-9)
    p.set_state(p.get_state())
    info = p.solve(1e-4, 200000)
    assert info["status"] == "OPTIMAL"
    x, y, _, _ = p.result()
    assert o.eval_unscaled(x, y)["rel_kkt"] <= 1e-4 * (1 + 1e-6)
