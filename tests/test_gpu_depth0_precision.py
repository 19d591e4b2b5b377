"""Arithmetic of depth 0 from bit planes: the FP64 re-evaluations it reports
are those of the per-depth test kernel, and where the statistic is FP64 from
the start (by the options, or from 5e8 pair-samples on) there are none.

The counts are whole numbers; a wide band keeps every pair's p-value far (many
times the FP32 error) from the band's ends.
"""

import numpy as np
import pytest

from bnsynth import make_dataset

pytestmark = pytest.mark.gpu

TESTS, PAIRS = 1, 2  # options.depth0: the per-depth test kernel, the contraction


@pytest.fixture(scope="module")
def bns():
    import paper_2212_04259_amd as b
    b.load()
    return b


def _data(k):
    return make_dataset(16 + 7 * k, 20 + 7 * k, 3, 2, 5, 0.5, 700 + 900 * k, seed=8100 + k)


def _rechecks(bns, sets, alphas, **opt):
    hs = [bns.bns_dataset_create(d.data, d.cards) for d in sets]
    o = bns.bns_options_default(recheck_band=0.3, **opt)
    if len(hs) == 1:
        outs = [bns.bns_pc_skeleton_dataset(hs[0], alphas[0], 1, o)]
    else:
        outs = bns.bns_pc_skeleton_batch(hs, alphas, [1] * len(hs), o)
    return [s.stats[0]["rechecks"] for s in outs]


@pytest.mark.parametrize("statistic,df_rule", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("datasets", [1, 3])
def test_rechecks_are_reported(bns, statistic, df_rule, datasets):
    sets = [_data(k) for k in range(datasets)]
    alphas = [0.05, 0.4, 0.9][:datasets]
    print(f"depth 0 rechecks stat={statistic} df={df_rule} datasets={datasets}", flush=True)
    want = _rechecks(bns, sets, alphas, depth0=TESTS, statistic=statistic, df_rule=df_rule)
    assert min(want) > 10
    assert _rechecks(bns, sets, alphas, statistic=statistic, df_rule=df_rule) == want


@pytest.mark.parametrize("opt", [dict(precision=1), dict(depth0=PAIRS), dict(precision=1, depth0=PAIRS), dict(precision=1, statistic=1, df_rule=1)])
def test_fp64_statistic(bns, opt):
    print(f"depth 0 in FP64 {opt}", flush=True)
    assert _rechecks(bns, [_data(2)], [0.05], **opt) == [0]


@pytest.mark.parametrize("m,fp64", [(19_000, False), (21_000, True)])
def test_fp64_by_work(bns, m, fp64):
    # 225 variables: 25,200 pairs, 5e8 pair-samples at 19,842 samples
    n = 225
    rng = np.random.default_rng(m)
    data, cards = rng.integers(0, 3, (n, m), dtype=np.uint8), np.full(n, 3, dtype=np.uint8)
    print(f"depth 0 of {n} x {m}", flush=True)
    ds = bns.bns_dataset_create(data, cards)
    sk = bns.bns_pc_skeleton_dataset(ds, 0.05, 1, bns.bns_options_default(recheck_band=0.3))
    assert (sk.stats[0]["rechecks"] == 0) == fp64


@pytest.mark.parametrize("band,alpha", [(0.0, 0.05), (1e-6, 1e-4), (1e-3, 1e-3)])
def test_rechecks_at_the_ends_of_the_band(bns, band, alpha):
    # a narrow band, and an alpha no larger than it: with alpha = band a pair
    # whose p is 0 to the last bit of alpha is not within the band
    ds = make_dataset(60, 80, 3, 2, 4, 0.5, 6_000, seed=8200)
    h = bns.bns_dataset_create(ds.data, ds.cards)
    print(f"depth 0 rechecks band={band} alpha={alpha}", flush=True)
    got, want = [bns.bns_pc_skeleton_dataset(h, alpha, 1, bns.bns_options_default(recheck_band=band, **opt)).stats[0]["rechecks"]
                 for opt in (dict(), dict(depth0=TESTS))]
    # (a pair whose p is at an end of the band to the FP32 error may fall on either side)
    assert abs(got - want) <= 1


def _span(bns, h, alpha, depth):
    o = bns.bns_options_default(depth0=0)
    return float(np.median([bns.bns_pc_skeleton_dataset(h, alpha, 1, o).stats[depth]["span_seconds"] for _ in range(25)]))


def test_small_alpha_costs_no_more_than_its_fp64(bns):
    # alpha below the band: every dependent decision is made again in FP64
    ds = make_dataset(20, 25, 3, 2, 4, 0.5, 5_000, seed=8301)
    h = bns.bns_dataset_create(ds.data, ds.cards)
    print("depths 0 and 1 at a small alpha", flush=True)
    for depth, most in ((0, 2.0), (1, 2.0)):
        usual, small = _span(bns, h, 0.05, depth), _span(bns, h, 1e-4, depth)
        print(f"depth {depth}: {usual * 1e6:.1f} us at 0.05, {small * 1e6:.1f} us at 1e-4", flush=True)
        assert small < most * usual
