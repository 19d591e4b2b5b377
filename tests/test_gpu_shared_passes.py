"""Deep depths, whose instance shares a test's passes among its units: no slower
than the instance without (the same search with constant two-category columns
added, which take part in depth 0 only and lower the mean cardinality that
decides), and with the same tests; and the oracle's results where Y has many
categories and a pass few strata.
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


def _stats(bns, data, cards, depth, alpha, **opt):
    h = bns.bns_dataset_create(data, cards)
    o = bns.bns_options_default(**opt)
    runs = [bns.bns_pc_skeleton_dataset(h, alpha, depth, o).stats[depth] for _ in range(15)]
    return float(np.median([s["span_seconds"] for s in runs])), runs[0]["tests_required"]


def _columns(cards, m, seed):
    """Independent columns of skewed categories: at a high alpha most edges
    reach the last depth."""
    rng = np.random.default_rng(seed)
    cols = [rng.choice(r, m, p=np.arange(1, r + 1) / (r * (r + 1) / 2)) for r in cards]
    return np.array(cols, dtype=np.uint8), np.array(cards, dtype=np.uint8)


def _both(bns, edges, hi, m, seed, depth, alpha=0.05):
    ds = make_dataset(60, edges, 3, 2, hi, 0.5, m, seed=seed)
    return _compare_spans(bns, ds.data, ds.cards, depth, alpha, f"up to {hi} categories", pad=180)


def _compare_spans(bns, data, cards, depth, alpha, label, pad, **opt):
    n, m = data.shape
    print(f"depth {depth} of {n} x {m}, {label}", flush=True)
    shared, tests = _stats(bns, data, cards, depth, alpha, **opt)
    more = np.zeros((pad, m), np.uint8), np.full(pad, 2, np.uint8)
    alone, tests2 = _stats(bns, np.concatenate([data, more[0]]), np.concatenate([cards, more[1]]), depth, alpha, **opt)
    assert tests == tests2 > 0
    print(f"{tests} tests: {shared * 1e6:.1f} us, without shared passes {alone * 1e6:.1f} us", flush=True)
    return shared, alone


def test_six_columns(bns):
    shared, alone = _both(bns, 78, 8, 50_000, 4, 4)
    assert shared < 1.1 * alone


@pytest.mark.parametrize("edges,hi,seed,depth", [(78, 5, 9, 5), (90, 4, 13, 6), (90, 6, 14, 6), (90, 6, 15, 5)])
def test_few_tests(bns, edges, hi, seed, depth):
    # 7 to 24 tests, 26 chunks of samples each
    shared, alone = _both(bns, edges, hi, 130_000, seed, depth)
    assert shared < 1.15 * alone


@pytest.mark.parametrize("edges,hi,m,seed,depth", [(90, 6, 130_000, 18, 5), (78, 8, 50_000, 3, 4)])
def test_small_alpha(bns, edges, hi, m, seed, depth):
    # alpha below the re-check band: nearly every decision is made in FP64
    shared, alone = _both(bns, edges, hi, m, seed, depth, alpha=1e-4)
    assert shared < alone


WIDE_Y = [[5, 200, 5, 5, 5, 5], [3, 60, 3, 3, 3, 3, 3], [2, 100, 2, 2, 40, 2, 2], [5, 7, 5, 5, 7, 5, 7]]


@pytest.mark.parametrize("cards", WIDE_Y, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("opt", [dict(), dict(recheck_band=0.0), dict(recheck_band=0.5), dict(precision=1), dict(test_group=1),
                                 dict(statistic=1, df_rule=1), dict(statistic=1, df_rule=1, recheck_band=0.0)], ids=str)
def test_wide_y(bns, orc, cards, opt):
    if "test_group" in opt and cards == WIDE_Y[2]:
        pytest.skip("a stratum of 100 x 40 cells is larger than a wave's share of the LDS")
    data, c = _columns(cards, 6_001, seed=sum(cards))
    print(f"wide Y {cards} {opt}", flush=True)
    alpha = 0.9
    ref = orc.pc_skeleton(data, c, alpha, -1, statistic=opt.get("statistic", 0), df_rule=opt.get("df_rule", 0))
    o = bns.bns_options_default(split_min_samples=1024, **opt)
    compare_with_oracle(bns.bns_pc_skeleton(data, c, alpha, -1, o), ref, f"{cards} {opt}")


@pytest.mark.parametrize("cards,depth", [(WIDE_Y[0], 3), (WIDE_Y[1], 4)], ids=str)
def test_few_strata(bns, cards, depth):
    data, c = _columns(cards, 100_001, seed=1)
    shared, alone = _compare_spans(bns, data, c, depth, 0.9995, f"cards {cards}", 60, split_min_samples=1024, statistic=1,
                                   df_rule=1)
    assert shared < alone


def test_large_alpha(bns):
    # alpha within the re-check band of 1
    data, c = _columns([3, 60, 3, 3, 3, 3, 3], 100_001, seed=1)
    shared, alone = _compare_spans(bns, data, c, 5, 0.9995, "alpha 0.9995", 60, split_min_samples=1024)
    assert shared < alone
