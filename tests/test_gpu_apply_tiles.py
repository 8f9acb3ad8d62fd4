"""K u and the residual over the tiles of levels from 97 nodes wide: tile edges along
x and y (exact, 2^n + 1, ragged), shallow z chunks, cubic cells and not.  The public
Apply gives K u at displacement nodes too.  A stencil value is a sum of some 150
terms of the size of |K| |u|, in another order than the oracle's: 1e-13 of the
largest value."""
import numpy as np
import pytest
import torch

import oracle
from _util import random_problem, rel_max, say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncell", [(96, 24, 4), (97, 30, 3), (127, 33, 5), (128, 32, 16),
                                   (192, 24, 6), (199, 41, 7), (256, 32, 12)])
def test_apply_and_residual(ncell):
    from paper_2212_02362_amd import Solver
    p = random_problem(ncell, seed=5, floor=1e-3, cubic=sum(ncell) % 2 == 0)
    say("apply over tiles", ncell)
    S = Solver(p.ncell, p.h)
    S.set_problem_from(p)
    rng = np.random.default_rng(6)
    u = rng.standard_normal((3,) + tuple(n + 1 for n in reversed(ncell)))
    psi = oracle.floor_psi(p.psi_raw, p.psi_floor)
    Ku = oracle.apply(p.ncell, p.h, p.lam, p.mu, psi, u)
    out = torch.full(u.shape, float("nan"), dtype=torch.float64, device="cuda")
    assert rel_max(to_np(S.apply(u, out)), Ku) <= 1e-13
    assert rel_max(to_np(S.level_apply(0, u)), Ku) <= 1e-13
    mask, _ = oracle.dirichlet(p.ncell, p.kind, p.val)
    f = to_np(S.rhs()[0])
    ref = np.where(np.asarray(mask).reshape(u.shape) != 0, 0.0, f - Ku)
    r, norm = S.residual(u)
    assert np.abs(to_np(r) - ref).max() <= 1e-13 * (np.abs(f).max() + np.abs(Ku).max())
    assert abs(norm - np.linalg.norm(ref)) <= 1e-12 * norm
    assert S.residual(u, want_r=False)[1] == norm
