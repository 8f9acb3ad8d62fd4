"""Displacement nodes without solid around them (psi_floor 0 and a void cell at the corner
of a clamped face: a zero diagonal that no free DOF has) on levels wide enough for the
tiled kernels.  Such a node keeps its prescribed value and the solve follows the oracle's:
FP64 histories to 1e-9, a mixed cycle's (an FP32 correction) to 1e-4, as on split rows."""
import numpy as np
import pytest

import oracle
from _util import rel_l2, say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("krylov", [0, 1])
@pytest.mark.parametrize("corner", [(0, 0, 0), (-1, -1, 0), (-1, 0, 0)])
@pytest.mark.parametrize("ncell", [(192, 32, 16), (208, 32, 16)])
def test_void_corner_of_a_clamped_face(ncell, corner, krylov, precision):
    from paper_2212_02362_amd import Solver
    say("zero diagonal", ncell, corner, "krylov", krylov, "precision", precision)
    rng = np.random.default_rng(3)
    psi = rng.uniform(0.2, 1.0, tuple(reversed(ncell)))
    psi[corner] = 0.0
    kind, val = np.zeros((6, 3), np.int32), np.zeros((6, 3))
    kind[0, :] = 1
    val[1, 0] = 1e-3
    h, lam, mu = (1.0 / ncell[1],) * 3, 0.6, 0.4
    b = rng.standard_normal((3,) + tuple(n + 1 for n in reversed(ncell)))
    u_o, hist_o, _ = oracle.solve(ncell, h, lam, mu, psi, 0.0, kind, val, b, rtol=0.0,
                                  max_cycles=2, krylov=krylov)
    assert np.isfinite(hist_o).all()
    S = Solver(ncell, h, rtol=0.0, max_cycles=2, krylov=krylov, precision=precision)
    S.set_problem(psi, lam, mu, 0.0, kind, val, b)
    u, hist, _ = S.solve()
    tol = 1e-9 if precision == 0 else 1e-4
    assert np.all(np.abs(hist - hist_o) <= tol * hist_o), (hist, hist_o)
    if precision == 0:
        assert rel_l2(to_np(u), u_o) <= 1e-11, rel_l2(to_np(u), u_o)
