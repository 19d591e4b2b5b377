"""GPU parity of depth 1 from bit planes against the oracle: every pair of
plane counts of X and Y (cardinalities 2 to 5), sample counts at the edges of
the planes' words and of a lane's 16 bytes, edges whose tests take several
passes and segments, the other statistics and precision, several alphas in
one batch, and the routes that keep the test kernel.

Skeleton, removal depths, sepsets and per-depth counts are whole numbers and
equal the oracle's exactly.
"""

import numpy as np
import pytest

from bnsynth import make_dataset
from golden_util import compare_with_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bns():
    import paper_2212_04259_amd as b
    b.load()
    return b


def _chain(cards, m, seed, keep=0.75):
    """Columns that repeat the previous one's value in most samples: many
    edges survive depth 0, and their tests run over many ranks."""
    rng = np.random.default_rng(seed)
    cols = []
    for r in cards:
        c = rng.integers(0, r, m)
        if cols:
            k = rng.random(m) < keep
            c[k] = cols[-1][k] % r
        cols.append(c)
    return np.array(cols, dtype=np.uint8), np.array(cards, dtype=np.uint8)


PAIRS = 2  # options.depth0: small searches take the path too


def _compare(bns, orc, data, cards, alpha, max_depth, label, statistic=0, df_rule=0, **opt):
    print(label, flush=True)
    opt = dict(dict(depth0=PAIRS), **opt)
    ref = orc.pc_skeleton(data, cards, alpha, max_depth, statistic=statistic, df_rule=df_rule)
    o = bns.bns_options_default(statistic=statistic, df_rule=df_rule, **opt)
    got = bns.bns_pc_skeleton(data, cards, alpha, max_depth, o)
    compare_with_oracle(got, ref, label)
    return got


@pytest.mark.parametrize("m", [1, 31, 33, 127, 128, 129, 1023, 1025, 8191, 8193, 20_001])
def test_samples_at_word_edges(bns, orc, m):
    data, cards = _chain([2, 3, 4, 5, 2, 3, 4, 5, 3, 2], m, seed=m)
    _compare(bns, orc, data, cards, 0.05, 1, f"bits m={m}")


@pytest.mark.parametrize("rx", [2, 3, 4, 5])
@pytest.mark.parametrize("rz", [2, 5])
def test_plane_counts(bns, orc, rx, rz):
    # every (r_X, r_Y) with Z of two or five categories
    data, cards = _chain([rx, 2, rz, 3, rz, 4, rz, 5, rz, rx], 4_000, seed=10 * rx + rz)
    _compare(bns, orc, data, cards, 0.01, 1, f"bits rx={rx} rz={rz}")


@pytest.mark.parametrize("n", [2, 15, 16, 17, 63, 64, 65, 129])
def test_pair_blocks(bns, orc, n):
    # depth 0 in blocks of 16 x 16 pairs, 64-bit adjacency rows
    rng = np.random.default_rng(n)
    data, cards = _chain(rng.integers(1, 6, n).tolist(), 700, seed=n, keep=0.5)
    for max_depth in (0, 2):
        _compare(bns, orc, data, cards, 0.05, max_depth, f"bits n={n} depth<={max_depth}")


@pytest.mark.parametrize("n,r", [(30, 5), (40, 2), (70, 3)])
def test_many_ranks(bns, orc, n, r):
    # a dense skeleton: up to 2 (n - 2) tests per edge, passes of one test at r = 5
    rng = np.random.default_rng(n)
    h = rng.integers(0, r, 1_500)
    cols = [np.where(rng.random(1_500) < 0.7, h, rng.integers(0, r, 1_500)) for _ in range(n)]
    data, cards = np.array(cols, dtype=np.uint8), np.full(n, r, dtype=np.uint8)
    got = _compare(bns, orc, data, cards, 0.05, 1, f"bits dense n={n} r={r}")
    assert got.stats[1]["tests_required"] > 2 * got.stats[1]["edges"]


@pytest.mark.parametrize("statistic,df_rule,precision", [(0, 0, 1), (1, 0, 0), (0, 1, 0), (1, 1, 1)])
def test_other_statistics_and_fp64(bns, orc, statistic, df_rule, precision):
    for m in (60, 5_001):
        data, cards = _chain([5, 3, 4, 2, 5, 3, 4, 2, 3, 3, 5], m, seed=m + statistic)
        _compare(bns, orc, data, cards, 0.05, 1, f"bits stat={statistic} df={df_rule} fp64={precision} m={m}",
                 statistic, df_rule, precision=precision)


def test_batch_with_several_alphas(bns, orc):
    dss = [make_dataset(12 + 5 * k, 20 + 5 * k, 3, 2, 5, 0.5, 900 + 1_111 * k, seed=7000 + k) for k in range(5)]
    alphas = [0.05, 0.01, 0.2, 1e-4, 0.9995]
    hs = [bns.bns_dataset_create(d.data, d.cards) for d in dss]
    print("bits batch of alphas", flush=True)
    outs = bns.bns_pc_skeleton_batch(hs, alphas, [-1, 1, 2, -1, -1], bns.bns_options_default(depth0=PAIRS))
    for d, a, md, got in zip(dss, alphas, [-1, 1, 2, -1, -1], outs):
        compare_with_oracle(got, orc.pc_skeleton(d.data, d.cards, a, md), f"alpha={a}")


def test_wider_variables_and_limits_keep_the_test_kernel(bns, orc):
    # a variable of six categories, a workspace limit without room for the
    # pairwise tables, and options that fix depth 1's shape: the same results
    ds = make_dataset(20, 30, 3, 2, 6, 0.5, 3_000, seed=7100)
    assert ds.cards.max() == 6
    _compare(bns, orc, ds.data, ds.cards, 0.05, -1, "bits card 6")
    ds = make_dataset(20, 30, 3, 2, 4, 0.5, 3_000, seed=7200)
    for opt in (dict(block_depths=2), dict(group_tests=2), dict(depth0=1), dict(recheck_band=0.0),
                dict(recheck_band=0.5), dict(use_graph=0), dict(timing=1)):
        _compare(bns, orc, ds.data, ds.cards, 0.05, -1, f"bits {opt}", **opt)
