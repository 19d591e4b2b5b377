"""The routes of a search and of all pairs at the limits between them: a
workspace limit that leaves room for the pairwise tables, for the planes only
or for neither, the largest sample count that depth 1 takes from planes, and
planes of all pairs at the edges of words, blocks and tiles from the sample
count on that makes them worth it.

Skeletons, depths and sepsets are whole numbers and equal; statistics of all
pairs agree with the oracle's to 1e-9 (exact counts, FP64 terms).
"""

import numpy as np
import pytest
import torch

from bnsynth import make_dataset
from golden_util import compare_with_oracle
from test_gpu_planes import _check

pytestmark = pytest.mark.gpu

TESTS, PAIRS = 1, 2  # options.depth0
E_NOMEM = 4


@pytest.fixture(scope="module")
def bns():
    import paper_2212_04259_amd as b
    b.load()
    return b


def _route(sk):
    """Whether depth 1 ran from planes (its work units are edges' segments, not
    ranks; of many edges), and the samples per chunk of depth 0's contraction (0: the test
    kernel)."""
    s0, s1 = sk.stats[0], sk.stats[1]
    return s1["tickets"] < s1["tests_required"], s0["chunk_samples"] if s0["test_group"] == 3 else 0


def test_limit_between_tables_and_planes(bns, orc):
    # pairwise tables of 1.4 M words (5.6 MiB); planes 0.6 MiB; 4,200 samples:
    # the contraction's chunks are whole blocks of planes
    ds = make_dataset(300, 330, 3, 4, 4, 0.5, 4_200, seed=8701)
    assert ds.cards.min() == 4
    want = orc.pc_skeleton(ds.data, ds.cards, 0.05, 2)
    h = bns.bns_dataset_create(ds.data, ds.cards)
    routes, refused = [], 0
    for mb in list(range(20, 72)) + [0]:
        o = bns.bns_options_default(depth0=PAIRS, workspace_mb=mb)
        try:
            got = bns.bns_pc_skeleton_dataset(h, 0.05, 2, o)
        except bns.BnsError as e:
            assert e.status == E_NOMEM and not routes, f"{mb} MiB refused, less accepted"
            refused += 1
            continue
        r = _route(got)
        if not routes or routes[-1][0] != r:
            print(f"from {mb} MiB: depth 1 from planes {r[0]}, depth-0 chunks {r[1]}", flush=True)
            compare_with_oracle(got, want, f"limit {mb} MiB")
            routes.append((r, mb))
    assert refused > 0
    assert [r[0] for r, _ in routes] == [False, True]  # without the tables first, then with them
    assert all(r[1] % 1024 == 0 for r, _ in routes)


def test_limit_between_planes_and_bytes(bns):
    # eight planes a variable take as much as its bytes: 128 MiB of planes
    n, m = 8, 1 << 24
    gen = torch.Generator(device="cuda").manual_seed(8702)
    data = torch.randint(0, 9, (n, m), generator=gen, device="cuda", dtype=torch.uint8)
    data[1] = torch.where(torch.rand(m, generator=gen, device="cuda") < 0.01, data[0], data[1])
    torch.cuda.synchronize()
    ds = bns.bns_dataset_wrap_device(data, m, np.full(n, 9, np.uint8))
    seen = {}
    for mb in (100, 0):
        print(f"all pairs and search of {n} x {m}, limit {mb} MiB", flush=True)
        o = bns.bns_options_default(depth0=PAIRS, workspace_mb=mb)
        pairs = bns.bns_ci_pairs(ds, 0.05, o)
        sk = bns.bns_pc_skeleton_dataset(ds, 0.05, 1, o)
        seen[mb] = (sk.stats[0], pairs, sk)
    assert seen[100][0]["test_group"] == seen[0][0]["test_group"] == 3
    assert seen[100][0]["chunk_samples"] % 1024 != 0 and seen[0][0]["chunk_samples"] % 1024 == 0  # of bytes, of planes
    for key in ("stat", "df", "p"):
        assert np.array_equal(np.asarray(seen[100][1][key]), np.asarray(seen[0][1][key])), key
    a, b = seen[100][2], seen[0][2]
    assert (a.adj == b.adj).all() and (a.depth == b.depth).all() and a.sepsets == b.sepsets
    assert b.adj[0, 1] == 1


@pytest.mark.parametrize("m", [(1 << 26) - 1, 1 << 26])
def test_most_samples_from_planes(bns, m):
    n = 4
    ld = (m + 15) // 16 * 16
    gen = torch.Generator(device="cuda").manual_seed(8703)
    data = torch.zeros((n, ld), dtype=torch.uint8, device="cuda")
    data[0, :m] = torch.randint(0, 5, (m,), generator=gen, device="cuda", dtype=torch.uint8)
    for v in range(1, n):
        own = torch.randint(0, 5, (m,), generator=gen, device="cuda", dtype=torch.uint8)
        data[v, :m] = torch.where(torch.rand(m, generator=gen, device="cuda") < 0.002, data[v - 1, :m], own)
    torch.cuda.synchronize()
    ds = bns.bns_dataset_wrap_device(data, m, np.full(n, 5, np.uint8))
    out = []
    for opt in (dict(), dict(depth0=TESTS, precision=1)):
        print(f"{n} x {m} {opt}", flush=True)
        out.append(bns.bns_pc_skeleton_dataset(ds, 0.05, 2, bns.bns_options_default(**opt)))
    a, b = out
    assert (a.adj == b.adj).all() and (a.depth == b.depth).all() and a.sepsets == b.sepsets
    assert [s["tests_required"] for s in a.stats] == [s["tests_required"] for s in b.stats]
    assert len(a.stats) > 1


@pytest.mark.parametrize("m", [4_095, 4_096, 4_097, 4_127, 4_129, 5_119, 5_120, 5_121, 6_143, 6_145])
def test_all_pairs_from_planes_at_word_and_block_edges(bns, orc, m):
    _check(bns, orc, [2, 3, 4, 5, 6, 9, 2, 1, 3], m, seed=m)


@pytest.mark.parametrize("cards", [[1, 1, 1], [1, 2], [8, 9, 1, 2], [2] * 65])
def test_all_pairs_from_planes_few_categories(bns, orc, cards):
    _check(bns, orc, cards, 4_500, seed=3, sample=200)
