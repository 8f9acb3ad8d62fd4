"""The bottom's inverse in FP64 cycles against the bottom CG that it stands for (a cap
on the CG's iterations, here never reached, keeps the CG): bottoms of one node to the
largest that takes it and one past it, 2D and 3D, V-cycles and CG, a second problem and
changed options on one context.  Both solve the bottom to 1e-12 of its load, so the
histories of a few cycles agree to 1e-9 and follow the oracle's."""
import numpy as np
import pytest

import oracle
from _util import random_problem, rel_l2, say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("krylov", [0, 1])
@pytest.mark.parametrize("ncell", [(4, 4), (24, 40), (48, 8), (38, 34), (8, 8, 8), (24, 12, 12), (28, 20, 12),
                                   (24, 20, 16), (28, 28, 24), (44, 10, 6), (30, 28, 20), (28, 28, 28), (52, 44)])
def test_inverse_follows_cg(ncell, krylov):
    from paper_2212_02362_amd import Solver
    say("bottom inverse", ncell, "krylov", krylov)
    S = Solver(ncell, tuple(1.0 / n for n in ncell), rtol=0.0, max_cycles=4, krylov=krylov)
    for seed in (21, 22):
        p = random_problem(ncell, seed=seed, floor=1e-3, cubic=False)
        p.h = S.h
        S.set_options(bottom_max_iter=0)
        S.set_problem_from(p)
        u, hist, _ = S.solve()
        _, hist_o, _ = oracle.solve(p.ncell, p.h, p.lam, p.mu, p.psi_raw, p.psi_floor, p.kind,
                                    p.val, p.b, rtol=0.0, max_cycles=4, krylov=krylov)
        S.set_options(bottom_max_iter=100000)
        v, hist_c, _ = S.solve()
        assert np.all(np.abs(hist - hist_c) <= 1e-9 * hist_c), (hist, hist_c)
        assert np.all(np.abs(hist - hist_o) <= 1e-9 * hist_o), (hist, hist_o)
        assert rel_l2(to_np(u), to_np(v)) <= 1e-9


def test_inverse_is_that_of_the_problem():
    """Options that change the bottom, mixed precision in between, a new problem."""
    from paper_2212_02362_amd import Solver
    ncell = (24, 12, 12)
    say("bottom inverse: options and problems in turn")
    S = Solver(ncell, (1.0 / 12,) * 3, rtol=1e-10, max_cycles=300)
    ps = [random_problem(ncell, seed=s, floor=1e-2, cubic=True) for s in (1, 2)]
    for p in ps:
        p.h = S.h
    ref = [oracle.solve(p.ncell, p.h, p.lam, p.mu, p.psi_raw, p.psi_floor, p.kind, p.val, p.b,
                        rtol=1e-10, max_cycles=300)[0] for p in ps]
    for k, opts in ((0, {}), (1, dict(precision=1)), (1, dict(precision=0)), (0, {}),
                    (0, dict(bottom_rtol=1e-3)), (1, dict(bottom_rtol=1e-12))):
        S.set_options(**opts)
        S.set_problem_from(ps[k])
        u, _, st = S.solve()
        assert st == 0 and rel_l2(to_np(u), ref[k]) <= 1e-7, (k, opts)
