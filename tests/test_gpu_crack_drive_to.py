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
