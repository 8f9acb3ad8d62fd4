"""Device memory a context asks for: the arrays that its solves hold at once, and the
bottom's solution operator only where the options at creation can use it."""
import ctypes
import math

import pytest


def _bytes(ncell, **opts):
    from paper_2212_02362_amd import _lib
    L = _lib.lib()
    g, o = _lib.SbmGrid(), _lib.SbmOptions()
    g.dim = len(ncell)
    for a in range(3):
        g.ncell[a] = ncell[a] if a < g.dim else 0
        g.h[a] = 1.0
    L.sbm_default_options(ctypes.byref(o))
    for k, v in opts.items():
        setattr(o, k, v)
    return L.sbm_workspace_bytes(ctypes.byref(g), ctypes.byref(o)), L.sbm_num_levels(ctypes.byref(g))


@pytest.mark.parametrize("ncell", [(256, 256, 256), (128, 128, 128), (192, 96, 96), (28, 28, 28)])
def test_vectors_of_the_hierarchy(ncell):
    """psi in both precisions and three vectors in each per level, five more on the finest."""
    got, nlev = _bytes(ncell, precision=1)
    want = 0
    for l in range(nlev):
        nc = [n >> l for n in ncell]
        nodes = math.prod(n + 1 for n in nc)
        want += 12 * math.prod(nc) + 3 * 3 * 12 * nodes + (5 * 3 * 8 * nodes if l == 0 else 0)
    assert want <= got <= want * 1.01 + 200_000, (got, want)


def test_bottom_operator_only_where_it_can_be_used():
    full = _bytes((28, 28, 28))[0]
    for opts in (dict(precision=1), dict(bottom_rtol=1e-6), dict(bottom_max_iter=50)):
        assert full - _bytes((28, 28, 28), **opts)[0] == 1536 * 1536 * 8
    assert _bytes((256, 256, 256))[0] - _bytes((256, 256, 256), precision=1)[0] <= 200_000
