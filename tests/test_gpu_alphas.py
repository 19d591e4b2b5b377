"""A search's cost does not depend on whether its alpha was used before, nor on
how many alphas a batch has."""

import time

import numpy as np
import pytest

from bnsynth import make_dataset

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bns():
    import paper_2212_04259_amd as b
    b.load()
    return b


def _seconds(f, calls):
    t = []
    for k in range(calls + 3):
        t0 = time.perf_counter()
        f(k)
        t.append(time.perf_counter() - t0)
    return float(np.median(t[3:]))


def test_new_alpha(bns):
    ds = make_dataset(20, 25, 3, 2, 4, 0.5, 5_000, seed=8301)
    h = bns.bns_dataset_create(ds.data, ds.cards)
    o = bns.bns_options_default()

    def call(alpha):
        bns.free_skeleton(bns.skeleton_handle(h, alpha, -1, o))

    print("new alphas", flush=True)
    same = _seconds(lambda k: call(0.05), 60)
    new = _seconds(lambda k: call(0.05 + 1e-7 * (k + 1)), 60)
    print(f"same alpha {same * 1e6:.1f} us, new alpha {new * 1e6:.1f} us", flush=True)
    assert new < 1.5 * same  # (1.9 with a table of 127 pairs of quantiles made anew)


def test_many_alphas(bns):
    dss = [make_dataset(20, 25, 3, 2, 4, 0.5, 5_000, seed=8400 + k) for k in range(100)]
    hs = [bns.bns_dataset_create(d.data, d.cards) for d in dss]
    o = bns.bns_options_default()

    def call(alphas):
        for s in bns.skeleton_batch_handles(hs, alphas, [-1] * len(hs), o):
            bns.free_skeleton(s)

    print("a batch of 100 alphas", flush=True)
    one = _seconds(lambda k: call([0.05] * 100), 12)
    own = _seconds(lambda k: call([0.05 + 1e-5 * j for j in range(100)]), 12)
    print(f"one alpha {one * 1e6:.0f} us, 100 alphas {own * 1e6:.0f} us", flush=True)
    assert own < 3 * one  # (10 with such a table for each)
