"""Sums that the host waits for in pinned memory: solves on two threads with a stream
each, one after another, and with live timing (which synchronises the stream instead)
give the same numbers bit for bit."""
import threading

import numpy as np
import pytest
import torch

from _util import random_problem, say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("krylov", [0, 1])
def test_waits_of_two_threads(krylov, precision):
    from paper_2212_02362_amd import Solver
    say("host sums", krylov, precision)
    ps = [random_problem(n, seed=s, floor=1e-2, cubic=True)
          for n, s in (((16, 16, 16), 3), ((64, 48), 4))]

    def run(p, stream, timed=False):
        with torch.cuda.stream(stream):
            S = Solver(p.ncell, p.h, rtol=0.0, max_cycles=12, krylov=krylov, precision=precision)
            S.profile(timed)
            S.set_problem_from(p)
            out = []
            for _ in range(3):
                u, hist, _ = S.solve()
                out.append((to_np(u), hist))
            return out

    ref = [run(p, torch.cuda.Stream()) for p in ps]
    got = [None, None]

    def work(k, stream):
        got[k] = run(ps[k], stream)
    ts = [threading.Thread(target=work, args=(k, torch.cuda.Stream())) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(2):
        for a, b in zip(ref[k] + ref[k], got[k] + run(ps[k], torch.cuda.Stream(), timed=True)):
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
