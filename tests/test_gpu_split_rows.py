"""Solves whose wide levels have split rows (even columns of a row first, then the
odd ones): ragged and exact tiles along x and y, chunks of few planes, one to
three sweeps, FP64 and mixed.  The workspace is filled with NaN first: the colour
half-sweep writes one colour per buffer, so the other half of a row may not have
been written when it is read past the box.  FP64 runs follow the oracle's first
cycles to 1e-9 in rho and 1e-11 in u (rounding of two cycles, as the wide-grid
trajectory test); a mixed cycle is an FP32 correction of relative accuracy 2^-24
per operation, a few hundred of them: 1e-4 of each residual."""
import numpy as np
import pytest

import oracle
from _util import random_problem, rel_l2, say, to_np

pytestmark = pytest.mark.gpu

GRIDS = [(96, 32, 16), (128, 32, 16), (104, 48, 16), (192, 40, 8), (256, 32, 16)]


def _solve(p, **opts):
    from paper_2212_02362_amd import Solver
    S = Solver(p.ncell, p.h, rtol=0.0, max_cycles=2, **opts)
    S._ws.fill_(255)  # NaN in every vector
    S.set_problem_from(p)
    u, hist, _ = S.solve()
    return to_np(u), hist


@pytest.mark.parametrize("krylov", [0, 1])
@pytest.mark.parametrize("nu", [1, 2, 3])
@pytest.mark.parametrize("ncell", GRIDS)
def test_split_rows_follow_the_oracle(ncell, nu, krylov):
    p = random_problem(ncell, seed=11, floor=1e-3, cubic=sum(ncell) % 3 != 0)
    say("split rows", ncell, "nu", nu, "krylov", krylov)
    u_o, hist_o, _ = oracle.solve(p.ncell, p.h, p.lam, p.mu, p.psi_raw, p.psi_floor, p.kind,
                                  p.val, p.b, rtol=0.0, max_cycles=2, nu_pre=nu, nu_post=nu,
                                  krylov=krylov)
    u, hist = _solve(p, nu_pre=nu, nu_post=nu, krylov=krylov)
    assert np.all(np.abs(hist - hist_o) <= 1e-9 * hist_o)
    assert rel_l2(u, u_o) <= 1e-11, rel_l2(u, u_o)
    um, histm = _solve(p, nu_pre=nu, nu_post=nu, krylov=krylov, precision=1)
    assert np.isfinite(um).all() and np.all(np.abs(histm - hist_o) <= 1e-4 * hist_o)


def test_solve_rhs_and_warm_start_on_split_rows():
    from paper_2212_02362_amd import Solver
    p = random_problem((128, 32, 16), seed=12, floor=1e-2, cubic=True)
    say("split rows: adjoint solve, warm start, options changed between solves")
    S = Solver(p.ncell, p.h, rtol=1e-10, max_cycles=200)
    S._ws.fill_(255)
    S.set_problem_from(p)
    u, hist, st = S.solve()
    assert st == 0
    _, again, st = S.solve(u0=u)
    assert st == 0 and len(again) == 1
    for opts in (dict(precision=1), dict(krylov=1), dict(precision=0), dict(smoother=1, krylov=0)):
        S.set_options(**opts)
        v, _, st = S.solve(u0=u)  # converged whatever rows the options choose
        assert st == 0 and rel_l2(to_np(v), to_np(u)) <= 1e-12
    S.set_options(smoother=0)
    fA, fB = S.rhs()
    x, _, st = S.solve_rhs(fB)  # K x = fA - K uD on the free DOF: x is the free part of u
    assert st == 0
    free = to_np(S.residual(u * 0.5)[0]) != 0.0
    assert rel_l2(to_np(x)[free], to_np(u)[free]) <= 1e-7
