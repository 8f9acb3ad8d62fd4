"""Composite solves of one problem are the same bits, one after another and after the
options changed and came back (bottoms of the base level inside the tail and outside it)."""
import numpy as np
import pytest

import sbm_inputs as si
from _util import say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base", [12, 14])
def test_same_bits_adaptive(base):
    from paper_2212_02362_amd import AmrSolver
    say("repeated adaptive solves", base)
    p, psis = si.ellipsoidal_voids_amr(base=base, levels=2, block=4)
    S = AmrSolver(p.ncell, p.h, len(psis), 4, rtol=0.0, max_cycles=7)
    S.set_problem(psis, p.lam, p.mu, p.psi_floor, p.kind, p.val)
    u, hist, _ = S.solve()
    for change in ({}, dict(nu_pre=1), dict(precision=1)):
        if change:
            old = {k: getattr(S._opts, k) for k in change}
            S.set_options(**change)
            S.solve()
            S.set_options(**old)
        v, hist_v, _ = S.solve()
        assert np.array_equal(hist, hist_v), change
        assert all(np.array_equal(to_np(a), to_np(b)) for a, b in zip(u, v)), change
