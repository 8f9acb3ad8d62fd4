"""The bottom solve inside a cycle, measured by its own residual: a stiff part behind a
layer at the floor (a through crack), where a solution operator formed to a small updated
residual still misses by the contrast.  Without smoothing a cycle adds the prolongation of
the bottom's solution x to the iterate, so x is read back at the coincident nodes and its
load is the restricted residual before.  bottom_rtol 1e-12 bounds the residual of either
way to solve; forming both on the host adds rounding of 1e-15: 2e-12.  Bottoms inside the
one-workgroup tail (2D, 3D) and outside it, an early cycle and a later one."""
import numpy as np
import pytest

import oracle
from _util import say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("floor", [1e-3, 1e-6, 1e-9])
@pytest.mark.parametrize("ncell", [(10, 6), (10, 26), (10, 8, 8), (10, 10, 10), (14, 14, 14)])
def test_bottom_residual_behind_a_floor_layer(ncell, floor):
    from paper_2212_02362_amd import Solver
    d = len(ncell)
    rng = np.random.default_rng(0)
    raw = np.ones(tuple(reversed(ncell)))
    k = 2 * (ncell[0] // 4)
    raw[..., k:k + 2] = 0.0  # one layer of bottom cells
    kind, val = np.zeros((6, 3), np.int32), np.zeros((6, 3))
    kind[0, :d] = 1
    h, lam, mu = (1.0 / ncell[1],) * d, 0.6, 0.4
    psi = oracle.floor_psi(raw, floor)
    ut = rng.standard_normal((d,) + tuple(n + 1 for n in reversed(ncell)))
    ut[..., 0] = 0.0
    g = oracle.apply(ncell, h, lam, mu, psi, ut)
    g[..., 0] = 0.0
    nc2, h2 = tuple(n // 2 for n in ncell), tuple(2 * x for x in h)
    mask2 = oracle.dirichlet(nc2, kind, val)[0]
    psi2 = oracle.coarsen_psi(ncell, psi)

    def after(m):
        say("bottom residual", ncell, floor, m)
        S = Solver(ncell, h, rtol=0.0, max_cycles=m, nu_pre=0, nu_post=0)
        S.set_problem(raw, lam, mu, floor, kind, val)
        return to_np(S.solve_rhs(g)[0])
    for m in (1, 5):
        u0, u1 = after(m), after(m + 1)
        r = g - oracle.apply(ncell, h, lam, mu, psi, u0)
        r[..., 0] = 0.0
        f2 = oracle.restrict(ncell, r, mask2)
        x2 = (u1 - u0)[(slice(None),) + (slice(None, None, 2),) * d]
        r2 = f2 - oracle.apply(nc2, h2, lam, mu, psi2, x2)
        r2[..., 0] = 0.0
        res = np.linalg.norm(r2) / np.linalg.norm(f2)
        assert res <= 2e-12, (m, res)
