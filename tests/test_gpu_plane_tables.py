"""Which tests of depths 2 and more count from bit planes: tables that padding
to powers of two makes large stay with the bytes, and are counted there by the
loops of their number of columns.  Results equal the oracle's exactly."""

import numpy as np
import pytest

from bnsynth import make_dataset
from golden_util import compare_with_oracle

pytestmark = pytest.mark.gpu

PLANES_FROM = 1 << 17  # samples


@pytest.fixture(scope="module")
def bns():
    import paper_2212_04259_amd as b
    b.load()
    return b


def _chain(cards, m, seed, keep=0.6):
    """Each column repeats one of the two before it in most samples: edges that
    survive several depths."""
    rng = np.random.default_rng(seed)
    cols = []
    for r in cards:
        c = rng.integers(0, r, m)
        for prev in cols[-2:]:
            k = rng.random(m) < keep / 2
            c[k] = prev[k] % r
        cols.append(c)
    return np.array(cols, dtype=np.uint8), np.array(cards, dtype=np.uint8)


# bits of four to six columns from below 4 to above 9; padding from none (2, 4)
# to (8 / 5)^k and (4 / 3)^k; one-category variables
CARDS = [[2] * 9, [4] * 9, [5] * 8, [3] * 9, [5, 2, 5, 2, 2, 5, 2, 2, 5], [3, 5, 4, 2, 5, 3, 2, 4, 5], [1, 2, 3, 4, 5, 1, 5, 4, 3]]


@pytest.mark.parametrize("cards", CARDS, ids=lambda c: "".join(map(str, c)))
@pytest.mark.parametrize("m", [PLANES_FROM - 1, PLANES_FROM, PLANES_FROM + 33])
def test_tables(bns, orc, cards, m):
    data, cards = _chain(cards, m, seed=sum(cards) + m % 7)
    print(f"plane tables {cards.tolist()} m={m}", flush=True)
    ref = orc.pc_skeleton(data, cards, 0.01, 4)
    for opt in (dict(), dict(split_min_samples=-1), dict(test_group=1)):
        o = bns.bns_options_default(depth0=2, **opt)
        compare_with_oracle(bns.bns_pc_skeleton(data, cards, 0.01, 4, o), ref, f"{cards.tolist()} m={m} {opt}")


@pytest.mark.parametrize("statistic,df_rule,precision", [(1, 0, 0), (0, 1, 0), (1, 1, 0), (0, 0, 1), (1, 1, 1)])
@pytest.mark.parametrize("split", [0, -1])
def test_other_statistics(bns, orc, statistic, df_rule, precision, split):
    # a table padded to powers of two adds nothing to the statistic or the
    # adjusted df; a category and a stratum that no sample has, and a variable
    # of one category
    data, cards = _chain([3, 5, 4, 2, 5, 3, 1, 4], PLANES_FROM + 33, seed=11 + statistic)
    data[0][data[0] == 2] = 0
    data[4][(data[4] == 3) & (data[3] == 1)] = 1
    print(f"plane tables stat={statistic} df={df_rule} fp64={precision} split={split}", flush=True)
    ref = orc.pc_skeleton(data, cards, 0.01, 4, statistic=statistic, df_rule=df_rule)
    o = bns.bns_options_default(depth0=2, statistic=statistic, df_rule=df_rule, precision=precision, split_min_samples=split)
    got = bns.bns_pc_skeleton(data, cards, 0.01, 4, o)
    compare_with_oracle(got, ref, f"stat={statistic} df={df_rule} fp64={precision}")
    assert len(got.stats) > 3


@pytest.mark.parametrize("statistic,df_rule", [(0, 0), (1, 1)])
def test_long_and_short_datasets(bns, orc, statistic, df_rule):
    # the longest one decides for the batch
    sizes = [PLANES_FROM + 33, 1_000, 31, 20_001, 129]
    sets = [_chain([3, 5, 4, 2, 4, 3, 2, 5], m, seed=40 + k) for k, m in enumerate(sizes)]
    print("plane tables, long and short datasets", flush=True)
    hs = [bns.bns_dataset_create(d, c) for d, c in sets]
    o = bns.bns_options_default(depth0=2, statistic=statistic, df_rule=df_rule)
    outs = bns.bns_pc_skeleton_batch(hs, [0.01] * len(hs), [-1] * len(hs), o)
    for (d, c), m, got in zip(sets, sizes, outs):
        compare_with_oracle(got, orc.pc_skeleton(d, c, 0.01, -1, statistic=statistic, df_rule=df_rule), f"m={m}")


@pytest.mark.parametrize("seed", [3, 4])
def test_no_slower_than_from_bytes(bns, seed):
    # five columns of up to five categories: just below and just above the rule
    ds = make_dataset(60, 78, 3, 2, 5, 0.5, PLANES_FROM, seed=seed)
    span = []
    for m in (PLANES_FROM - 1, PLANES_FROM):
        print(f"depth 3 of 60 x {m}", flush=True)
        h = bns.bns_dataset_create(np.ascontiguousarray(ds.data[:, :m]), ds.cards)
        runs = [bns.bns_pc_skeleton_dataset(h, 0.05, 3).stats for _ in range(15)]
        span.append(float(np.median([s[3]["span_seconds"] for s in runs])))
    print(f"bytes {span[0] * 1e6:.1f} us, planes {span[1] * 1e6:.1f} us", flush=True)
    assert span[1] < 1.5 * span[0]  # (1.75 and 1.95 where every table was counted from planes)
