"""GPU parity of the depths of 2 and more that count from bit planes against
the oracle: tables at the edges of one pass (12 bits of cell index) and of the
16 shared passes, beyond them (the byte form), with variables of one category,
sample counts at the edges of words and of plane blocks, one test per wave and
per workgroup, samples and passes split over several units, the other
statistic, df rule and precision, and several datasets in one call.

Independent columns at a high alpha keep most edges to the last depth.
Skeleton, removal depths, sepsets and per-depth counts are whole numbers and
equal the oracle's exactly.
"""

import numpy as np
import pytest

from golden_util import compare_with_oracle

pytestmark = pytest.mark.gpu

PAIRS = 2  # options.depth0: small searches take the path too
ALPHA = 0.9995


@pytest.fixture(scope="module")
def bns():
    import paper_2212_04259_amd as b
    b.load()
    return b


def _columns(cards, m, seed):
    rng = np.random.default_rng(seed)
    # (skewed categories: cells of very different counts)
    cols = [rng.choice(r, m, p=np.arange(1, r + 1) / (r * (r + 1) / 2)) for r in cards]
    return np.array(cols, dtype=np.uint8), np.array(cards, dtype=np.uint8)


def _compare(bns, orc, data, cards, alpha, max_depth, label, statistic=0, df_rule=0, reach=None, **opt):
    print(label, flush=True)
    ref = orc.pc_skeleton(data, cards, alpha, max_depth, statistic=statistic, df_rule=df_rule)
    o = bns.bns_options_default(statistic=statistic, df_rule=df_rule, **dict(dict(depth0=PAIRS), **opt))
    got = bns.bns_pc_skeleton(data, cards, alpha, max_depth, o)
    compare_with_oracle(got, ref, label)
    if reach is not None:
        assert len(got.stats) > reach, "the depth under test was not reached"


# depth 6 has 8 bits of cell index (2s), 16 (3s and 4s: 16 passes of a test),
# 24 (5s: the byte form), and those between
@pytest.mark.parametrize("cards,m", [([2] * 8, 6_001), ([3] * 8, 6_001), ([4] * 8, 60_001), ([5] * 8, 120_001),
                                     ([2, 3, 4, 5, 3, 4, 2, 3], 20_001), ([2, 2, 2, 2, 2, 4, 4, 4], 6_001),
                                     ([4, 1, 2, 3, 1, 4, 3, 2, 2], 6_001)])
@pytest.mark.parametrize("split", [0, 1024])
def test_deep(bns, orc, cards, m, split):
    data, c = _columns(cards, m, seed=sum(cards))
    _compare(bns, orc, data, c, ALPHA, -1, f"deep {cards} split {split}", reach=5, split_min_samples=split)


@pytest.mark.parametrize("m", [4095, 4129, 8191, 8193, 10_271])
def test_deep_sample_edges(bns, orc, m):
    data, c = _columns([2, 3, 4, 2, 4, 3, 4, 4], m, seed=m)
    _compare(bns, orc, data, c, ALPHA, -1, f"deep m={m}", reach=5, split_min_samples=1024)


@pytest.mark.parametrize("m", [(1 << 17) - 1, 1 << 17, (1 << 17) + 1, 140_031])
@pytest.mark.parametrize("cards", [[2] * 5, [3, 3, 2, 4, 5], [4] * 5, [5] * 5])
def test_many_samples(bns, orc, cards, m):
    data, c = _columns(cards, m, seed=m + cards[0])
    _compare(bns, orc, data, c, ALPHA, -1, f"m={m} {cards}", reach=2)


@pytest.mark.parametrize("mask", [dict(wave_depths=0xFC), dict(block_depths=0xFC)])
def test_groups(bns, orc, mask):
    data, c = _columns([4, 3, 2, 5, 4, 3], (1 << 17) + 5, seed=3)
    _compare(bns, orc, data, c, ALPHA, -1, f"groups {mask}", reach=3, **mask)


@pytest.mark.parametrize("statistic,df_rule", [(1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("split", [0, 1024])
def test_other_statistics(bns, orc, statistic, df_rule, split):
    # (three samples per cell at depth 5: empty rows, columns and strata)
    data, c = _columns([4, 3, 4, 2, 4, 3, 4, 4], 20_001, seed=11)
    _compare(bns, orc, data, c, ALPHA, -1, f"stat {statistic} df {df_rule}", statistic=statistic, df_rule=df_rule, reach=5,
             split_min_samples=split)


def test_fp64(bns, orc):
    data, c = _columns([4, 3, 4, 2, 4, 3, 4, 4], 6_001, seed=5)
    _compare(bns, orc, data, c, ALPHA, -1, "fp64", reach=5, precision=1, split_min_samples=1024)


def test_batch(bns, orc):
    print("deep batch", flush=True)
    sets, refs = [], []
    for k, (cards, m) in enumerate([([4] * 8, 60_001), ([3] * 7, 8_193), ([2, 5, 4, 3, 4, 4, 2, 3], 20_001)]):
        data, c = _columns(cards, m, seed=k)
        refs.append(orc.pc_skeleton(data, c, ALPHA, -1))
        sets.append(bns.bns_dataset_create(data, c))
    o = bns.bns_options_default(depth0=PAIRS, split_min_samples=1024)
    for k, (got, ref) in enumerate(zip(bns.bns_pc_skeleton_batch(sets, [ALPHA] * 3, [-1] * 3, o), refs)):
        compare_with_oracle(got, ref, f"deep batch {k}")
