"""The crack driving force into an array of its own: the arithmetic of the update in
place, the input kept, a NaN history kept as in place."""
import ctypes

import pytest
import torch

from _util import random_problem, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncell", [(1, 1), (33, 18), (257, 64), (13, 9, 7)])
def test_crack_drive_into_other_array(ncell):
    from paper_2212_02362_amd import Solver
    from paper_2212_02362_amd._lib import lib
    say("crack drive out of place", ncell)
    p = random_problem(ncell, seed=3, floor=0.05, body=False, zero_frac=0.0)
    S = Solver(p.ncell, p.h)
    S.set_problem_from(p)
    g = torch.Generator(device="cuda").manual_seed(4)
    u = torch.randn((len(ncell),) + S.node_shape, generator=g, device="cuda", dtype=torch.float64)
    H0, _ = S.crack_drive(u, torch.zeros(S.cell_shape, device="cuda", dtype=torch.float64))
    H = H0 * 2 * torch.rand(S.cell_shape, generator=g, device="cuda", dtype=torch.float64)
    H.view(-1)[0] = float("nan")
    kept = H.clone()
    Hn, intact = S.crack_drive(u, H)
    same = lambda a, b: torch.equal(a.view(torch.int64), b.view(torch.int64))
    assert same(H, kept) and torch.isnan(Hn.view(-1)[0])
    Hi, intact_i = S.crack_drive(u, H, inplace=True)
    assert Hi is H and same(Hn, H) and torch.equal(intact, intact_i)
    P = lambda t: ctypes.c_void_p(t.data_ptr())
    for h, o, i in ((H, u, intact), (H, Hn, H), (H, Hn, Hn)):
        assert lib().sbm_crack_drive_to(S._ctx, P(u), P(h), P(o), P(i)) == -1


@pytest.mark.parametrize("scale", [1.0, 1e-5, 1e-140])
def test_principal_strains(scale):
    """Uniform strains: diagonal, with equal values, of rank one, nearly diagonal,
    random.  Corner differences and the rotations err by a few ulp of the largest
    entry: 1e-13 of the energy of the strain's norm."""
    import numpy as np

    from paper_2212_02362_amd import Solver
    n = (2, 2, 2)
    S = Solver(n, (1.0,) * 3)
    lam, mu = 0.6, 0.4
    S.set_problem(np.ones(n), lam, mu, 1e-3, np.array([[1] * 3] + [[0] * 3] * 5), np.zeros((6, 3)))
    rng = np.random.default_rng(1)
    one = np.ones((3, 3))
    cases = [np.zeros((3, 3)), np.diag([1.0, -2.0, 3.0]), np.eye(3), one, -one,
             np.eye(3) + 1e-9 * one, np.diag([1.0, 1e-9, 0.0]) + 1e-20 * one,
             np.array([[0.0, 1.0, 0.0], [1.0, 0.0, 0.0], [0.0, 0.0, 0.0]]),
             np.array([[0.0, 0.0, 1e-12], [0.0, 1.0, 0.0], [1e-12, 0.0, 0.0]])]
    cases += [m + m.T for m in rng.standard_normal((8, 3, 3))]
    x = np.stack(np.meshgrid(*[np.arange(3.0)] * 3, indexing="ij")[::-1])
    for k, E in enumerate(cases):
        say("principal strains", k, scale)
        H, intact = S.crack_drive(np.tensordot(scale * E, x, 1), np.zeros(n))
        e = np.linalg.eigvalsh(E)
        p, m = np.maximum(e, 0), np.minimum(e, 0)
        wp, wm = (0.5 * lam * v.sum() ** 2 + mu * (v ** 2).sum() for v in (p, m))
        tol = 1e-13 * (lam + mu) * (E ** 2).sum()
        assert np.abs(H.cpu().numpy() / scale ** 2 - wp).max() <= tol, (k, wp)
        if abs(wp - wm) > 2 * tol:
            assert (intact.cpu().numpy() == (wp < wm)).all(), k
