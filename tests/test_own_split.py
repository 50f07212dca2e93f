"""The run table of the library's own split (column_runs with `fit`, the default
of every 3D batch), called in the library as built: every plane of every patch
in exactly one run along the +z links, no more runs than chains or resident
work-groups, a chain's share rounded down, FD runs shorter than a patch where
there are fewer patches than work-groups."""
import ctypes as C

import numpy as np
import pytest

import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I


class _Vec(C.Structure):   # std::vector<int4>
    _fields_ = [("begin", C.c_void_p), ("end", C.c_void_p), ("cap", C.c_void_p)]


def own_runs(kind, p, nbr, w, cus):
    f = pb.lib()._ZN2pb11column_runsEiiPKiS1_iib   # pb::column_runs(kind, K, p, nbr, w, cus, fit)
    f.restype = None
    f.argtypes = [C.POINTER(_Vec), C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_bool]
    p, nbr = np.ascontiguousarray(p, np.int32), np.ascontiguousarray(nbr, np.int32)
    v = _Vec()
    f(C.byref(v), kind, len(p), p.ctypes.data, nbr.ctypes.data, w, cus, True)
    n = (v.end - v.begin) // 16
    return np.array((C.c_int32 * (4 * n)).from_address(v.begin)).reshape(n, 4)   # (copied; the vector is not freed)


def check(p, nbr, runs, pmin):
    count = [np.zeros(q, int) for q in p]
    for k, z, n, _ in runs:
        assert n >= 1
        for i in range(n):
            count[k][z] += 1
            z += 1
            if z == p[k] and i + 1 < n:
                s = nbr[k][5]
                assert nbr[s][4] == k and p[s] == p[k] >= pmin
                k, z = s, 0
    for c in count:
        np.testing.assert_array_equal(c, 1)


@pytest.mark.parametrize("grid,p,w", [((16, 16, 8), 16, 3), ((1, 1, 1), 16, 3), ((7, 5, 3), 11, 6), ((16, 16, 12), 8, 8),
                                      ((11, 9, 7), 13, 4), ((10, 10, 10), 16, 3), ((40, 40, 1), 9, 6)])
def test_grids(grid, p, w):
    K = int(np.prod(grid))
    ps, nbr = np.full(K, p, np.int32), I.periodic_grid(grid)
    runs = own_runs(0, ps, nbr, w, 256)
    check(ps, nbr, runs, 2)
    chains, planes = grid[0] * grid[1], grid[2] * p
    per = max(1, min(planes, w * 256 // chains))
    assert len(runs) == chains * per
    assert runs[:, 2].max() - runs[:, 2].min() <= 1
    if chains <= w * 256:
        assert len(runs) <= w * 256


@pytest.mark.parametrize("K", [1, 100, 383, 385, 500, 767, 768, 769, 3000])
def test_independent_patches(K):
    """between half and all of the work-groups: one run per patch, the split
    that a batch had before there was an own one"""
    ps, nbr = np.full(K, 16, np.int32), I.self_periodic(K, 3)
    runs = own_runs(0, ps, nbr, 3, 256)
    check(ps, nbr, runs, 2)
    assert len(runs) == K * max(1, min(16, 768 // K))


def test_mixed_sizes_and_fd():
    ps = np.array([16, 7, 3, 12, 5, 1, 16, 9, 4], np.int32)
    nbr = I.self_periodic(len(ps), 3)
    check(ps, nbr, own_runs(0, ps, nbr, 3, 256), 2)
    check(ps, nbr, own_runs(0, ps, nbr, 3, 2), 2)
    # Euler FD: a single patch is dealt to as many work-groups as it has planes
    one = own_runs(1, [16], I.self_periodic(1, 3), 2, 256)
    check([16], I.self_periodic(1, 3), one, 4)
    assert len(one) == 16
    g = I.periodic_grid((4, 4, 4))
    ps = np.full(64, 16, np.int32)
    runs = own_runs(1, ps, g, 2, 256)
    check(ps, g, runs, 4)
    assert len(runs) == 512 and np.all(runs[:, 2] == 2)
