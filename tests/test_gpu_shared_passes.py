"""Deep depths, whose instance shares a test's passes among its units: no slower
than the instance without (the same search with constant two-category columns
added, which take part in depth 0 only and lower the mean cardinality that
decides), and with the same tests.
"""

import numpy as np
import pytest

from bnsynth import make_dataset

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bns():
    import paper_2212_04259_amd as b
    b.load()
    return b


def _stats(bns, data, cards, depth, alpha):
    h = bns.bns_dataset_create(data, cards)
    runs = [bns.bns_pc_skeleton_dataset(h, alpha, depth).stats[depth] for _ in range(15)]
    return float(np.median([s["span_seconds"] for s in runs])), runs[0]["tests_required"]


def _both(bns, edges, hi, m, seed, depth, alpha=0.05):
    n = 60
    ds = make_dataset(n, edges, 3, 2, hi, 0.5, m, seed=seed)
    print(f"depth {depth} of {n} x {m}, up to {hi} categories", flush=True)
    shared, tests = _stats(bns, ds.data, ds.cards, depth, alpha)
    pad = np.zeros((3 * n, m), np.uint8), np.full(3 * n, 2, np.uint8)
    alone, tests2 = _stats(bns, np.concatenate([ds.data, pad[0]]), np.concatenate([ds.cards, pad[1]]), depth, alpha)
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
