"""The plastic load of columns of several nodes per thread (63 nodes per wave: rows
shorter than, equal to and longer than a wave; column lengths 1 to 10, cut short at the
top), and the radial return into arrays of its own.  A load value is a sum of some 100
products, known to about 1e-13 of the largest; the return out of place makes the
arithmetic of the return in place."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from _util import random_problem, rel_max, say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncell", [(1, 1, 1), (5, 3, 2), (62, 62, 3), (63, 60, 40),
                                   (130, 125, 70), (256, 129, 83)])
def test_source_columns(ncell):
    from paper_2212_02362_amd import Solver
    say("plastic source columns", ncell)
    p = random_problem(ncell, seed=8, floor=0.05, body=False, zero_frac=0.0)
    S = Solver(p.ncell, p.h)
    S.set_problem_from(p)
    ep = np.random.default_rng(9).standard_normal((6,) + tuple(reversed(ncell)))
    out = torch.full((3,) + S.node_shape, float("nan"), dtype=torch.float64, device="cuda")
    ref = oracle.plastic_source(p.ncell, p.h, p.lam, p.mu, oracle.floor_psi(p.psi_raw, 0.05), ep)
    assert rel_max(to_np(S.plastic_source(ep, out)), ref) <= 1e-13


def test_return_map_into_other_arrays():
    from paper_2212_02362_amd import Solver
    from paper_2212_02362_amd._lib import SbmJ2, lib
    say("return map out of place")
    p = random_problem((21, 14, 9), seed=3, floor=0.05, body=False)
    S = Solver(p.ncell, p.h)
    S.set_problem_from(p)
    g = torch.Generator(device="cuda").manual_seed(4)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.float64)
    u, ep, bt = 1e-2 * rand(3, *S.node_shape), 1e-2 * rand(6, *S.cell_shape), rand(6, *S.cell_shape)
    al = rand(*S.cell_shape).abs()
    kept = [t.clone() for t in (ep, al, bt)]
    new = S.return_map(u, ep, al, bt, 0.8, 0.1, 0.4)
    assert all(torch.equal(a, b) for a, b in zip((ep, al, bt), kept))
    old = S.return_map(u, ep, al, bt, 0.8, 0.1, 0.4, inplace=True)
    assert 0 < new[3] < al.numel() and old[0] is ep
    assert all(torch.equal(a, b) for a, b in zip(new[:3], old[:3])) and new[3] == old[3]
    P = lambda t: ctypes.c_void_p(t.data_ptr())
    m, e2, a2 = SbmJ2(1.0, 0.0, 1.0), torch.empty_like(ep), torch.empty_like(al)
    for outs in ((bt, a2, e2), (e2, ep, bt), (e2, a2, e2), (u, a2, bt)):
        assert lib().sbm_return_map_to(S._ctx, P(u), ctypes.byref(m), P(ep), P(al), P(bt),
                                       *map(P, outs), None) == -1
