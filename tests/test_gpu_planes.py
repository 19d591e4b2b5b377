"""GPU parity of the pair contraction from bit planes against the oracle at
the edges of its words (32 samples), blocks (1,024 samples) and tiles (64
planes), for tables completed in registers (up to 5 categories) and in loops,
for one-category variables, and for the byte form that wide variables keep.

Tolerances: the counts are exact and the statistic is formed in FP64 from
them, so statistics and p agree with the oracle's to 1e-9.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bns():
    import paper_2212_04259_amd as b
    b.load()
    return b


def _columns(cards, m, seed):
    """Columns that depend on one another: each repeats the previous one's
    value (modulo its own categories) in most samples."""
    rng = np.random.default_rng(seed)
    cols = []
    for r in cards:
        c = rng.integers(0, r, m)
        if cols:
            keep = rng.random(m) < 0.6
            c[keep] = cols[-1][keep] % r
        cols.append(c)
    return np.array(cols, dtype=np.uint8), np.array(cards, dtype=np.uint8)


def _check(bns, orc, cards, m, seed, sample=None, **opt):
    data, cards = _columns(cards, m, seed)
    print(f"planes m={m} planes={int(cards.sum()) - len(cards)} {opt}", flush=True)
    h = bns.bns_dataset_create(data, cards)
    r = bns.bns_ci_pairs(h, 0.05, bns.bns_options_default(**opt))
    idx = range(len(r["pairs"]))
    if sample is not None and sample < len(r["pairs"]):
        idx = np.random.default_rng(seed).choice(len(r["pairs"]), size=sample, replace=False)
    for q in idx:
        i, j = r["pairs"][q]
        s, df, p = orc.ci_test(data, cards, i, j, (), statistic=opt.get("statistic", 0),
                               df_rule=opt.get("df_rule", 0))
        assert r["df"][q] == df, (i, j)
        assert abs(r["stat"][q] - s) <= 1e-9 * max(abs(s), 1.0), (i, j, r["stat"][q], s)
        assert abs(r["p"][q] - p) <= 1e-9 * max(p, 1e-300) + 1e-15, (i, j, r["p"][q], p)


@pytest.mark.parametrize("m", [1, 31, 32, 33, 1023, 1024, 1025, 4096, 4097, 8193])
def test_samples_at_word_and_block_edges(bns, orc, m):
    _check(bns, orc, [2, 3, 4, 5, 6, 9, 2, 1, 3], m, seed=m)


@pytest.mark.parametrize("planes", [1, 63, 64, 65, 129])
def test_planes_at_tile_edges(bns, orc, planes):
    cards = [2, 1] if planes == 1 else [3] * (planes // 2) + [2] * (planes % 2)
    _check(bns, orc, cards, 5_000, seed=planes, sample=200)


@pytest.mark.parametrize("statistic,df_rule", [(0, 0), (1, 1)])
def test_mixed_cardinalities(bns, orc, statistic, df_rule):
    _check(bns, orc, [5, 6, 4, 17, 2, 1, 8, 255, 3], 20_011, seed=9, statistic=statistic, df_rule=df_rule)


def test_one_category_only(bns, orc):
    _check(bns, orc, [1, 1, 1], 100, seed=3)


def test_wide_variables_keep_the_byte_form(bns, orc):
    # 1,592 planes of 400,000 samples: 80 MB, above 64 MiB and the columns' 3.2 MB
    _check(bns, orc, [200] * 8, 400_000, seed=4)
