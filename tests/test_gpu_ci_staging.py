"""GPU test of the ways a CI batch's results reach the host: written by the
kernel itself (up to 256 tests), brought by a copying kernel (staging of
1 MiB), or copied from library buffers (beyond it).  The tests, the kernel
and its arithmetic are the same, so every result is equal bit for bit,
whatever the batch it was part of and whichever entry point ran it.
"""

import numpy as np
import pytest

from bnsynth import make_dataset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 4, 5, 255, 256, 257, 1_000, 23_000, 26_000])
def test_results_do_not_depend_on_the_batch(count):
    import paper_2212_04259_amd as bns
    ds = make_dataset(20, 25, 3, 2, 4, 0.5, 700, seed=8100)
    h = bns.bns_dataset_create(ds.data, ds.cards)
    rng = np.random.default_rng(count)
    tests = []
    for _ in range(count):
        v = rng.permutation(20)[:2 + int(rng.integers(0, 4))]
        tests.append((int(v[0]), int(v[1]), tuple(int(z) for z in v[2:])))
    print(f"staging count={count}", flush=True)
    whole = bns.bns_ci_batch(h, tests, 0.05)
    again = bns.bns_ci_batch_noalloc(h, tests, 0.05)
    step = 100 if count <= 1_000 else 5_000
    for key in ("g2", "df", "p", "flags"):
        assert np.array_equal(whole[key], again[key]), key
    for a in range(0, count, step):
        part = bns.bns_ci_batch(h, tests[a:a + step], 0.05)
        for key in ("g2", "df", "p", "flags"):
            assert np.array_equal(whole[key][a:a + step], part[key]), (key, a)


def test_outputs_may_be_null_and_calls_may_run_side_by_side():
    import ctypes
    import threading
    import paper_2212_04259_amd as bns
    ds = make_dataset(20, 25, 3, 2, 4, 0.5, 5_000, seed=8200)
    h = bns.bns_dataset_create(ds.data, ds.cards)
    tests = [(i, j, ()) for i in range(20) for j in range(i + 1, 20)]
    ref = bns.bns_ci_batch(h, tests, 0.05)
    rec = np.array([(x, y, 0, 0) for x, y, _ in tests], dtype=np.int32)
    p = np.zeros(len(tests))
    vp = ctypes.c_void_p
    o = bns.bns_options_default()
    st = bns.load().bns_ci_batch_noalloc(h.handle, rec.ctypes.data_as(vp), len(tests), None, 0, 0.05, ctypes.byref(o),
                                         None, None, p.ctypes.data_as(vp), None)
    assert st == 0 and np.array_equal(p, ref["p"])
    bad = []

    def work(call):
        for _ in range(50):
            r = call(h, tests, 0.05)
            if not np.array_equal(r["p"], ref["p"]):
                bad.append(call.__name__)

    ts = [threading.Thread(target=work, args=(c,)) for c in (bns.bns_ci_batch, bns.bns_ci_batch_noalloc,
                                                             bns.bns_ci_batch)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
