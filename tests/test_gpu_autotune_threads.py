"""The autotuner while another thread searches on the same device: what it
learns of its own searches does not come from the other's."""

import threading

import numpy as np
import pytest

from bnsynth import make_dataset
from golden_util import compare_with_oracle

pytestmark = pytest.mark.gpu


def test_concurrent_searches(orc):
    import paper_2212_04259_amd as bns
    bns.load()
    ds = make_dataset(24, 30, 3, 2, 4, 0.5, 3_000, seed=8601)
    other = make_dataset(20, 25, 3, 6, 6, 0.5, 2_000, seed=8602)  # (six categories: not from bit planes)
    h, h2 = bns.bns_dataset_create(ds.data, ds.cards), bns.bns_dataset_create(other.data, other.cards)
    want = orc.pc_skeleton(other.data, other.cards, 0.05, 1)
    done, bad = threading.Event(), []

    def search():
        while not done.is_set():
            got = bns.bns_pc_skeleton_dataset(h2, 0.05, 1)
            if not np.array_equal(got.adj, np.asarray(want.adj)):
                bad.append(got)

    t = threading.Thread(target=search)
    print("autotune beside another thread's searches", flush=True)
    t.start()
    try:
        # (a fixed replication cap: a key no other test tunes)
        best = bns.bns_autotune([h], [0.05], [-1], bns.bns_options_default(max_replicas=8), trials=1)
    finally:
        done.set()
        t.join()
    assert not bad
    # depths 0 and 1 run from bit planes: no wave or workgroup is chosen for them
    assert (best.wave_depths | best.block_depths) & 3 == 0
    compare_with_oracle(bns.bns_pc_skeleton_dataset(h, 0.05, -1, best), orc.pc_skeleton(ds.data, ds.cards, 0.05, -1), "tuned")
