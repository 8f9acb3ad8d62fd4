"""The load of an FP32 cycle is scaled into FP32's range whatever the starting residual's
size: a start far off (its residual 1e45 times the load's) contracts as a near one, up to
FP32 rounding (1e-4); and a nearly converged start in other units (stiffness 2^77 times
larger: powers of two commute with every rounding that neither overflows nor underflows)
gives the same bits."""
import numpy as np
import pytest

from _util import random_problem, say, to_np

pytestmark = pytest.mark.gpu


def _mixed(p, u0, cycles):
    from paper_2212_02362_amd import Solver
    S = Solver(p.ncell, p.h, rtol=0.0, max_cycles=cycles, precision=1)
    S.set_problem_from(p)
    u, hist, _ = S.solve(u0=u0)
    return to_np(u), hist


@pytest.mark.parametrize("ncell", [(192, 32, 16), (128, 32, 16)])
def test_start_far_off(ncell):
    p = random_problem(ncell, seed=2, floor=1e-2, cubic=True)
    v = np.random.default_rng(1).standard_normal((3,) + tuple(n + 1 for n in reversed(ncell)))
    hist = []
    for s in (1e6, 1e45):
        say("mixed scale, start", ncell, s)
        hist.append(_mixed(p, s * v, 3)[1])
        assert np.isfinite(hist[-1]).all()
    a, b = (h / h[0] for h in hist)
    assert np.all(np.abs(a - b) <= 1e-4 * a), (a, b)


@pytest.mark.parametrize("ncell", [(192, 32, 16), (128, 32, 16)])
def test_units(ncell):
    from paper_2212_02362_amd import Solver
    p = random_problem(ncell, seed=2, floor=1e-2, cubic=True)
    p.val[p.kind == 0] = 0.0  # (a traction would scale by another power)
    S = Solver(p.ncell, p.h, rtol=1e-10, max_cycles=300)
    S.set_problem_from(p)
    u0, _, st = S.solve()
    assert st == 0
    say("mixed scale, units", ncell)
    u, hist = _mixed(p, u0, 2)
    p.lam, p.mu, p.h, p.b = p.lam * 2.0 ** 37, p.mu * 2.0 ** 37, tuple(x * 2.0 ** -20 for x in p.h), p.b * 2.0 ** 77
    w, hist_w = _mixed(p, u0, 2)
    assert np.array_equal(hist, hist_w), (hist, hist_w)
    assert np.array_equal(u, w)
