"""Mixed V-cycle iteration on tiled finest levels, where the convergence test
writes the FP32 cycle's load (ragged tiles, cubic and non-cubic cells, a warm
start, a zero load).  The last entry of the history is the FP64 residual of the
returned u, so the oracle's residual of it agrees to FP64 rounding (1e-12 of
the load); the history follows the FP64 iteration's to the rounding of an FP32
cycle (2^-24 per operation, a few hundred of them: 1e-4 relative)."""
import numpy as np
import pytest

import oracle
from _util import random_problem, say, solver_for, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cubic", [False, True])
@pytest.mark.parametrize("ncell", [(192, 32, 16), (208, 48, 32)])
def test_mixed_vcycles_on_tiled_level(ncell, cubic):
    p = random_problem(ncell, seed=3, floor=1e-3, cubic=cubic)
    say("mixed tiled V-cycles", ncell, cubic)
    S = solver_for(p, precision=1, rtol=0.0, max_cycles=20)
    u, hist, _ = S.solve()
    psi = oracle.floor_psi(p.psi_raw, p.psi_floor)
    fA, fB, _ = oracle.rhs(p.ncell, p.h, p.lam, p.mu, psi, p.kind, p.val, p.b)
    mask, _ = oracle.dirichlet(p.ncell, p.kind, p.val)
    r = oracle.residual(p.ncell, p.h, p.lam, p.mu, psi, mask, to_np(u), fA)
    assert abs(np.linalg.norm(r) / np.linalg.norm(fB[mask == 0]) - hist[-1]) <= 1e-12
    _, hist64, _ = solver_for(p, precision=0, rtol=0.0, max_cycles=20).solve()
    assert np.all(np.abs(hist - hist64) <= 1e-4 * hist64 + 1e-13)
    _, warm, _ = S.solve(u0=u)  # goes on where the first solve stopped
    assert abs(warm[0] - hist[-1]) <= 1e-12 and warm[-1] < hist[-1]
    S.set_options(rtol=1e-10)
    x, _, st = S.solve_rhs(np.zeros(u.shape))  # zero load
    assert st == 0 and not to_np(x).any()
