"""GPU parity of all-pairs tests around the sample count from which the
contraction takes bit planes, at the edges of their words and blocks, for
tables completed in the lane's LDS (up to 8 categories) and in loops.

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


@pytest.mark.parametrize("statistic,df_rule", [(0, 0), (1, 1)])
@pytest.mark.parametrize("m", [33, 4095, 4096, 4127, 4129, 5119, 5121])
def test_pairs_around_the_forms(bns, orc, m, statistic, df_rule):
    print(f"pairs m={m} statistic {statistic} df {df_rule}", flush=True)
    rng = np.random.default_rng(m)
    cards = np.array([8, 2, 9, 7, 1, 3, 8, 4, 5, 6], dtype=np.uint8)
    data = np.array([rng.integers(0, r, m) for r in cards], dtype=np.uint8)
    keep = rng.random(m) < 0.5
    data[6, keep] = data[0, keep]
    h = bns.bns_dataset_create(data, cards)
    r = bns.bns_ci_pairs(h, 0.05, bns.bns_options_default(statistic=statistic, df_rule=df_rule))
    for q, (i, j) in enumerate(r["pairs"]):
        s, df, p = orc.ci_test(data, cards, i, j, (), statistic=statistic, df_rule=df_rule)
        assert r["df"][q] == df, (i, j)
        assert abs(r["stat"][q] - s) <= 1e-9 * max(abs(s), 1.0), (i, j, r["stat"][q], s)
        assert abs(r["p"][q] - p) <= 1e-9 * max(p, 1e-300) + 1e-15, (i, j, r["p"][q], p)
