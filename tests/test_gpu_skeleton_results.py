"""Results of a GPU search read through each accessor of its handle: the
adjacency, removal depths, separating sets one by one (before and after the
whole list, in both orders of a pair) and the CPDAG against the same skeleton
handed to bns_skeleton_create.  Variable counts around the eight pairs that
the orientation passes over at a time.  All whole numbers, equal exactly.
"""

import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bns():
    import paper_2212_04259_amd as b
    b.load()
    return b


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


@pytest.mark.parametrize("single_first", [False, True])
@pytest.mark.parametrize("n", [2, 7, 8, 9, 16, 25])
def test_accessors_agree(bns, n, single_first):
    print(f"accessors n={n}", flush=True)
    L = bns.load()
    rng = np.random.default_rng(n)
    cards = rng.integers(2, 4, n).astype(np.uint8)
    data = np.zeros((n, 3000), dtype=np.uint8)
    for i in range(n):
        data[i] = rng.integers(0, cards[i], 3000)
        if i:  # a copy of an earlier variable in most samples
            k = rng.random(3000) < 0.4
            data[i, k] = data[rng.integers(0, i), k] % cards[i]
    ds = bns.bns_dataset_create(data, cards)
    h = bns.skeleton_handle(ds, 0.05, -1, bns.bns_options_default())
    off, plen = np.empty((n, n), np.int64), ctypes.c_int64()
    if not single_first:
        assert L.bns_skeleton_removals(h, None, _p(off), None, 0, ctypes.byref(plen)) == 0
    adj, depth = np.empty((n, n), np.uint8), np.empty((n, n), np.int32)
    assert L.bns_skeleton_adjacency(h, _p(adj)) == 0
    assert L.bns_skeleton_removals(h, _p(depth), None, None, 0, None) == 0
    sets = {}
    for i in range(n):
        for j in range(n):
            if i == j:
                assert adj[i, j] == 0 and depth[i, j] == -1
                continue
            buf, ln, dd = np.full(n, -7, np.int32), ctypes.c_int32(), ctypes.c_int32()
            assert L.bns_skeleton_sepset(h, i, j, _p(buf), n, ctypes.byref(ln), ctypes.byref(dd)) == 0
            assert dd.value == depth[i, j] == ln.value and adj[i, j] == (dd.value < 0)
            if dd.value >= 0:
                sets[i, j] = tuple(int(v) for v in buf[:dd.value])
                assert list(sets[i, j]) == sorted(set(sets[i, j])) and i not in sets[i, j] and j not in sets[i, j]
            assert np.all(buf[max(dd.value, 0):] == -7)
    assert all(sets[j, i] == s for (i, j), s in sets.items())
    if single_first:
        assert L.bns_skeleton_removals(h, None, _p(off), None, 0, ctypes.byref(plen)) == 0
    assert np.array_equal(off >= 0, depth >= 0) and not off[depth == 0].any()
    assert plen.value == depth[np.triu(depth, 1) > 0].sum()
    ref = bns.collect(h, orient=True)
    assert np.array_equal(ref.adj, adj) and np.array_equal(ref.depth, depth)
    half = {k: s for k, s in sets.items() if k[0] < k[1]}
    assert ref.sepsets == half
    assert n < 9 or (any(half.values()) and adj.any())  # the case is not empty
    assert np.array_equal(ref.cpdag, bns.bns_orient(adj, half))
