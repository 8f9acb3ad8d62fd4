"""Solves of one problem, one after another and after the options changed and came back,
are the same bits: how the bottom is solved depends on the cycle, not on what ran before.
Bottoms inside the tail and outside it, split rows, V-cycles and CG, the adjoint entry (whose
load takes the place of the problem's in split rows) in between."""
import numpy as np
import pytest

from _util import random_problem, say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("krylov", [0, 1])
@pytest.mark.parametrize("ncell", [(16, 16, 16), (28, 28, 28), (56, 40, 48), (64, 48),
                                   (128, 32, 16)])
def test_same_bits(ncell, krylov):
    from paper_2212_02362_amd import Solver
    say("repeated solves", ncell, krylov)
    p = random_problem(ncell, seed=5, floor=1e-2, cubic=True)
    S = Solver(p.ncell, p.h, rtol=0.0, max_cycles=8, krylov=krylov)
    S.set_problem_from(p)
    u, hist, _ = S.solve()
    fB = S.rhs()[1]
    x, hist_x, _ = S.solve_rhs(fB)
    for change in ({}, dict(nu_pre=1), dict(precision=1), dict(bottom_rtol=1e-6)):
        if change:
            old = {k: S.options[k] for k in change}
            S.set_options(**change)
            S.solve()
            S.set_options(**old)
        v, hist_v, _ = S.solve()
        assert np.array_equal(hist, hist_v), change
        assert np.array_equal(to_np(u), to_np(v)), change
        y, hist_y, _ = S.solve_rhs(fB)
        assert np.array_equal(hist_x, hist_y) and np.array_equal(to_np(x), to_np(y)), change


@pytest.mark.parametrize("krylov", [0, 1])
@pytest.mark.parametrize("ncell,cycles", [((16, 16, 16), 1), ((16, 16, 16), 2), ((64, 48), 2),
                                          ((28, 28, 28), 6)])
def test_few_cycles_keep_the_cg(ncell, cycles, krylov):
    """Solves too short to earn back the bottom's inverse: the bits of the bottom CG (kept
    by a cap on its iterations that is never reached)."""
    from paper_2212_02362_amd import Solver
    say("few cycles", ncell, cycles, krylov)
    p = random_problem(ncell, seed=6, floor=1e-2, cubic=True)
    S = Solver(p.ncell, p.h, rtol=0.0, max_cycles=cycles, krylov=krylov)
    got = []
    for cap in (0, 100000):
        S.set_options(bottom_max_iter=cap)
        S.set_problem_from(p)
        for _ in range(2):
            u, hist, _ = S.solve()
            got.append((to_np(u), hist))
    for u, hist in got[1:]:
        assert np.array_equal(u, got[0][0]) and np.array_equal(hist, got[0][1])
