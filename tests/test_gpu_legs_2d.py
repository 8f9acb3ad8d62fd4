"""The legs of 2D FP64 V-cycles in one launch each: both tile sizes, exact and ragged
tiles, one and two sweeps on either leg (three stay with separate passes), V-cycles and
CG, mixed boundary tables, non-square cells, iterate and workspace full of NaN where
they start from zero.  The values are those of the separate passes up to rounding:
histories follow the oracle's first cycles to 1e-9, as on wide 3D grids."""
import numpy as np
import pytest

import oracle
from _util import random_problem, rel_l2, say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("krylov", [0, 1])
@pytest.mark.parametrize("nu", [(1, 1), (1, 2), (2, 1), (2, 2), (3, 2)])
@pytest.mark.parametrize("ncell", [(64, 64), (96, 40), (132, 68), (40, 200), (30, 510), (528, 512),
                                   (600, 480)])
def test_legs_follow_the_oracle(ncell, nu, krylov):
    from paper_2212_02362_amd import Solver
    say("2D legs", ncell, "nu", nu, "krylov", krylov)
    p = random_problem(ncell, seed=31, floor=1e-3, cubic=ncell[0] % 64 == 0)
    kw = dict(rtol=0.0, max_cycles=3, nu_pre=nu[0], nu_post=nu[1], krylov=krylov)
    u_o, hist_o, _ = oracle.solve(p.ncell, p.h, p.lam, p.mu, p.psi_raw, p.psi_floor, p.kind,
                                  p.val, p.b, **kw)
    S = Solver(p.ncell, p.h, **kw)
    S._ws.fill_(255)
    S.set_problem_from(p)
    u, hist, _ = S.solve()
    assert np.all(np.abs(hist - hist_o) <= 1e-9 * hist_o), (hist, hist_o)
    assert rel_l2(to_np(u), u_o) <= 1e-10
