"""The sensitivity of columns of several cells per thread: column lengths 1 to 16,
whole and cut short at the top, every chain rule, tractions on the faces.  A cell's
value is a sum of some 200 products of differences of corner values, so it is known to
about 1e-13 of the largest value."""
import numpy as np
import pytest
import torch

import oracle
from _util import random_problem, rel_max, say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncell", [(5, 3, 2), (64, 64, 131), (130, 125, 70), (256, 129, 83),
                                   (192, 160, 150)])
def test_columns(ncell):
    from paper_2212_02362_amd import Solver
    say("sensitivity columns", ncell)
    rng = np.random.default_rng(7)
    p = random_problem(ncell, seed=8, floor=0.05)
    shape = (3,) + tuple(n + 1 for n in reversed(ncell))
    u, lam = rng.standard_normal(shape), rng.standard_normal(shape)
    S = Solver(p.ncell, p.h)
    S.set_problem_from(p)
    g = oracle.sensitivity(p.ncell, p.h, p.lam, p.mu, p.kind, p.val, u, lam)
    assert rel_max(to_np(S.sensitivity(u, lam, lam_scale=0.5)), 0.5 * g) <= 1e-13
    raw = rng.uniform(0.0, 0.2, g.shape)
    got = S.sensitivity(u, lam, design=torch.tensor(raw, device="cuda"), chain=1)
    assert rel_max(to_np(got), np.where(raw > p.psi_floor, g, 0.0)) <= 1e-13
    rho = rng.uniform(0.0, 1.0, g.shape)
    got = S.sensitivity(u, lam, design=torch.tensor(rho, device="cuda"), chain=2)
    ref = np.where(rho ** 3 > p.psi_floor, 3.0 * rho ** 2 * g, 0.0)
    assert rel_max(to_np(got), ref) <= 1e-13
