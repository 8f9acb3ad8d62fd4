"""Small 3D levels whose sweeps are one launch: tiles exact and ragged along each axis,
one to three sweeps on either leg, V-cycles and CG, cubic cells and not, a workspace full
of NaN.  The values are those of the half-sweeps up to rounding: histories follow the
oracle's first cycles to 1e-9."""
import numpy as np
import pytest

import oracle
from _util import random_problem, rel_l2, say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("krylov", [0, 1])
@pytest.mark.parametrize("nu", [(1, 1), (2, 2), (3, 2), (2, 3), (1, 2)])
@pytest.mark.parametrize("ncell", [(32, 32, 32), (64, 64, 64), (44, 36, 52), (60, 28, 92),
                                   (128, 24, 40), (92, 32, 24)])
def test_sweeps_follow_the_oracle(ncell, nu, krylov):
    from paper_2212_02362_amd import Solver
    say("small sweeps", ncell, "nu", nu, "krylov", krylov)
    p = random_problem(ncell, seed=41, floor=1e-3, cubic=sum(ncell) % 3 != 0)
    kw = dict(rtol=0.0, max_cycles=3, nu_pre=nu[0], nu_post=nu[1], krylov=krylov)
    u_o, hist_o, _ = oracle.solve(p.ncell, p.h, p.lam, p.mu, p.psi_raw, p.psi_floor, p.kind,
                                  p.val, p.b, **kw)
    S = Solver(p.ncell, p.h, **kw)
    S._ws.fill_(255)
    S.set_problem_from(p)
    u, hist, _ = S.solve()
    assert np.all(np.abs(hist - hist_o) <= 1e-9 * hist_o), (hist, hist_o)
    assert rel_l2(to_np(u), u_o) <= 1e-10
