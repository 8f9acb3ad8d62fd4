"""fused_sweep = 1 on levels wider than 192 nodes: every Gauss-Seidel sweep of the finest
level is one launch, counted by live timing, in FP64 and mixed cycles; the iterates are
those of the half-sweeps up to rounding (FP64 1e-9 in rho; a mixed cycle, an FP32
correction, 1e-4).  Narrower levels keep their half-sweeps."""
import numpy as np
import pytest

from _util import random_problem, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("krylov", [0, 1])
@pytest.mark.parametrize("nu", [(2, 2), (1, 3)])
@pytest.mark.parametrize("ncell", [(192, 32, 16), (256, 32, 16), (128, 32, 16)])
def test_launches_and_iterates(ncell, nu, krylov, precision):
    from paper_2212_02362_amd import Solver
    say("fused option", ncell, nu, krylov, precision)
    p = random_problem(ncell, seed=9, floor=1e-3, cubic=True)
    hist, prof = [], []
    for fused in (0, 1):
        S = Solver(p.ncell, p.h, rtol=0.0, max_cycles=3, nu_pre=nu[0], nu_post=nu[1],
                   krylov=krylov, precision=precision, fused_sweep=fused)
        S.set_problem_from(p)
        hist.append(S.solve()[1])
        S.profile(True)
        assert np.array_equal(S.solve()[1], hist[-1])  # launch by launch: the same bits
        prof.append(S.profile_read())
        S.profile(False)
    assert np.all(np.abs(hist[0] - hist[1]) <= (1e-9 if precision == 0 else 1e-4) * hist[0])
    sweeps = sum(prof[1][k][1] for k in ("smooth", "sweep0", "smooth_dot"))
    cycles = 3 + krylov  # CG makes one more for the direction after the last
    if ncell[0] >= 192:
        assert sweeps == cycles * sum(nu), (prof[1], cycles)
    else:
        assert sweeps > cycles * sum(nu)
