"""The work that users of the library have it do, as measurable cases.

Kinds of case:
  ci      a batch of conditional-independence tests on a resident dataset
          (bns_ci_batch, bns_ci_batch_noalloc)
  pairs   every pairwise marginal test of a dataset (bns_ci_pairs)
  search  PC-stable on one resident dataset or on many in one call
          (bns_pc_skeleton_dataset, bns_pc_skeleton_batch), its skeleton,
          removal depths and CPDAG read back
  host    PC-stable from a host array, through the Python entry point

The calls go through the C ABI of include/bns.h as the package loads it, with
the caller's own arrays for the results, except in "host", which uses the
Python wrapper.  Data are samples of random Bayesian networks (random order,
bounded in-degree, Dirichlet CPT rows, forward sampling), the inputs the
method is for.
"""

import ctypes
import math

import numpy as np
import torch

import paper_2212_04259_amd as bns

MAX_DEPTHS = 24  # conditioning sets have at most 22 members
MAX_CI_WORK = 4096 * 50_000 * 4  # tests x samples x columns of the largest listed batch of tests


def listed():
    return [
        # one test on a small dataset: an interactive query, all latency
        dict(name="ci_one", kind="ci", n=20, m=5_000, card_hi=4, tests=1, nz_max=2, noalloc=False, fp64=False,
             x2=False, adjusted=False),
        # a serving loop's small batch through the allocation-free call, odd sample count
        dict(name="ci_small_noalloc", kind="ci", n=31, m=5_003, card_hi=4, tests=65, nz_max=2, noalloc=True,
             fp64=False, x2=False, adjusted=False),
        # a caller's own structure learner asks for thousands of tests at once
        dict(name="ci_batch", kind="ci", n=60, m=50_000, card_hi=4, tests=4096, nz_max=3, noalloc=False, fp64=False,
             x2=False, adjusted=False),
        # the other statistic, df rule and precision, wider variables, ragged sizes
        dict(name="ci_fp64_x2", kind="ci", n=37, m=49_999, card_hi=6, tests=777, nz_max=2, noalloc=False, fp64=True,
             x2=True, adjusted=True),
        # all pairwise tests of a few hundred variables (dependence screening)
        dict(name="pairs_500", kind="pairs", n=500, m=100_000, card_hi=4, x2=False, adjusted=False),
        # the smallest PC search in use: 20 variables, 5,000 rows
        dict(name="search_20", kind="search", n=20, m=5_000, card_hi=4, edge_ratio=1.25, alpha=0.05, max_depth=-1,
             datasets=1, wrap=False, x2=False, adjusted=False),
        # the 60-variable, 50,000-row network of the benchmark
        dict(name="search_60", kind="search", n=60, m=50_000, card_hi=4, edge_ratio=70 / 60, alpha=0.05,
             max_depth=-1, datasets=1, wrap=False, x2=False, adjusted=False),
        # the same scale with Pearson's X^2 and adjusted df, on a caller's device tensor, ragged
        dict(name="search_61_x2", kind="search", n=61, m=49_993, card_hi=4, edge_ratio=1.2, alpha=0.01, max_depth=-1,
             datasets=1, wrap=True, x2=True, adjusted=True),
        # 220 variables, 100,000 rows
        dict(name="search_220", kind="search", n=220, m=100_000, card_hi=5, edge_ratio=1.5, alpha=0.05, max_depth=-1,
             datasets=1, wrap=False, x2=False, adjusted=False),
        # the largest single network: 1,000 variables, 200,000 rows, bounded depth
        dict(name="search_1000", kind="search", n=1000, m=200_000, card_hi=4, edge_ratio=1.2, alpha=0.05, max_depth=4,
             datasets=1, wrap=True, x2=False, adjusted=False),
        # 64 datasets of 20 to 200 variables and 5,000 to 100,000 rows in one call
        dict(name="search_batch_64", kind="search", n=200, m=100_000, card_hi=5, edge_ratio=1.25, alpha=0.01,
             max_depth=-1, datasets=64, wrap=False, x2=False, adjusted=False),
        # from a NumPy array to skeleton, sepsets and CPDAG in Python
        dict(name="host_60", kind="host", n=60, m=50_000, card_hi=4, edge_ratio=70 / 60, alpha=0.05, max_depth=-1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ci", "ci", "pairs", "search", "search", "search", "batch", "host"])
    stat = dict(x2=rng.random() < 0.25, adjusted=rng.random() < 0.25)
    if kind == "ci":
        m = _log_int(rng, 1_000, 200_000)
        nz = rng.randint(0, 3)
        cap = max(1, MAX_CI_WORK // (m * (nz + 2)))
        return dict(kind="ci", n=rng.randint(20, 200), m=m, card_hi=rng.randint(3, 6),
                    tests=_log_int(rng, 1, min(8192, cap)), nz_max=nz, noalloc=rng.random() < 0.3,
                    fp64=rng.random() < 0.25, **stat)
    m = _log_int(rng, 2_000, 200_000)
    n = _log_int(rng, 20, 1000)
    if kind == "pairs":
        m = min(m, 100_000 * 500 * 500 // (n * n))
        return dict(kind="pairs", n=n, m=m, card_hi=rng.randint(3, 6), **stat)
    common = dict(card_hi=rng.randint(3, 5), edge_ratio=round(rng.uniform(1.0, 1.3), 3),
                  alpha=rng.choice([0.01, 0.05]))
    if kind == "host":
        return dict(kind="host", n=min(n, 100), m=m, max_depth=-1, **common)
    if kind == "batch":
        return dict(kind="search", n=min(n, 150), m=min(m, 80_000), max_depth=-1, datasets=rng.randint(2, 48),
                    wrap=False, **common, **stat)
    return dict(kind="search", n=n, m=m, max_depth=4 if n > 200 else -1, datasets=1, wrap=rng.random() < 0.5,
                **common, **stat)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _network(n, card_hi, edge_ratio, rng):
    """Random order, parents (at most 3 per variable), cardinalities 2..card_hi and CPTs (Dirichlet 0.5)."""
    order = rng.permutation(n)
    place = np.empty(n, dtype=np.int64)
    place[order] = np.arange(n)
    parents = [[] for _ in range(n)]
    left, tries = int(round(edge_ratio * n)), 0
    while left > 0 and tries < 100 * n:
        tries += 1
        a, b = (int(v) for v in rng.integers(0, n, 2))
        if a == b:
            continue
        p, c = (a, b) if place[a] < place[b] else (b, a)
        if p in parents[c] or len(parents[c]) >= 3:
            continue
        parents[c].append(p)
        left -= 1
    cards = rng.integers(2, card_hi + 1, n).astype(np.uint8)
    cum = []
    for v in range(n):
        cfg = int(np.prod([int(cards[p]) for p in parents[v]], dtype=np.int64)) if parents[v] else 1
        cum.append(np.cumsum(rng.dirichlet(np.full(int(cards[v]), 0.5), size=cfg), axis=1))
    return order, parents, cards, cum


def _sample(n, m, card_hi, edge_ratio, seed, ld=None):
    """Columns uint8 [n][ld] on the GPU (the first m of each row are samples) and the cardinalities."""
    rng = np.random.Generator(np.random.PCG64(seed))
    order, parents, cards, cum = _network(n, card_hi, edge_ratio, rng)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out = torch.zeros((n, ld or m), dtype=torch.uint8, device="cuda")
    width = int(max(cards))
    flat = torch.full((sum(len(c) for c in cum), width - 1), 2.0, dtype=torch.float32)
    first, at = [], 0
    for c in cum:
        flat[at:at + len(c), :c.shape[1] - 1] = torch.from_numpy(c[:, :-1].astype(np.float32))
        first.append(at)
        at += len(c)
    flat = flat.cuda()
    for v in order:
        v = int(v)
        u = torch.rand(m, generator=gen, device="cuda")
        cfg = torch.full((m,), first[v], dtype=torch.int64, device="cuda")
        stride = 1
        for p in parents[v]:
            cfg += out[p, :m].to(torch.int64) * stride
            stride *= int(cards[p])
        out[v, :m] = (u[:, None] >= flat[cfg]).sum(1).to(torch.uint8)
    torch.cuda.synchronize()
    return out, cards


def _tests(case, seed):
    """Random tests: x, y and up to nz_max conditioning variables, as the C ABI takes them."""
    rng = np.random.Generator(np.random.PCG64([seed, 1]))
    rec = np.zeros((case["tests"], 4), dtype=np.int32)
    pool = []
    for t in range(case["tests"]):
        nz = int(rng.integers(0, case["nz_max"] + 1)) if case["tests"] > 1 else case["nz_max"]
        v = rng.choice(case["n"], 2 + nz, replace=False)
        rec[t] = (v[0], v[1], nz, len(pool))
        pool.extend(int(z) for z in v[2:])
    return rec, np.asarray(pool or [0], dtype=np.int32), len(pool)


def _sizes(case):
    """(n, m) of every dataset of a search: the case's own, or n in [20, n], m in [m / 20, m]."""
    if case["datasets"] == 1:
        return [(case["n"], case["m"])]
    rng = np.random.Generator(np.random.PCG64([case["n"], case["m"], case["datasets"]]))
    ns = rng.integers(20, max(case["n"], 21) + 1, case["datasets"])
    ms = rng.integers(max(case["m"] // 20, 500), case["m"] + 1, case["datasets"])
    return list(zip(ns.tolist(), ms.tolist()))


def _options(case):
    return bns.bns_options_default(
        precision=bns.BNS_PREC_FP64 if case.get("fp64") else bns.BNS_PREC_FP32_RECHECK,
        statistic=bns.BNS_STAT_X2 if case.get("x2") else bns.BNS_STAT_G2,
        df_rule=bns.BNS_DF_ADJUSTED if case.get("adjusted") else bns.BNS_DF_DECLARED)


def _ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _ok(status):
    if status != bns._lib.BNS_OK:
        raise bns.BnsError(status, bns.load().bns_last_error().decode())


def prepare(case, seed):
    if case["kind"] == "host":
        data, cards = _sample(case["n"], case["m"], case["card_hi"], case["edge_ratio"], seed)
        return dict(case=case, data=data.cpu().numpy(), cards=cards)
    opt = _options(case)
    if case["kind"] == "search":
        sets = []
        for k, (n, m) in enumerate(_sizes(case)):
            ld = (m + 255) // 256 * 256 if case["wrap"] else None
            data, cards = _sample(n, m, case["card_hi"], case["edge_ratio"], seed * 1000 + k, ld)
            sets.append(bns.bns_dataset_wrap_device(data, m, cards) if case["wrap"]
                        else bns.bns_dataset_create(data.cpu().numpy(), cards))
        return dict(case=case, sets=sets, opt=opt, alphas=[case["alpha"]] * len(sets),
                    depths=[case["max_depth"]] * len(sets))
    data, cards = _sample(case["n"], case["m"], case["card_hi"], 1.25, seed)
    ds = bns.bns_dataset_create(data.cpu().numpy(), cards)
    state = dict(case=case, ds=ds, opt=opt)
    if case["kind"] == "ci":
        state["rec"], state["pool"], state["pool_len"] = _tests(case, seed)
    return state


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _statistics(count):
    return (np.empty(count, dtype=np.float64), np.empty(count, dtype=np.int64), np.empty(count, dtype=np.float64),
            np.empty(count, dtype=np.int32))


def _skeletons(L, handles, sets):
    """Adjacency, removal depths and CPDAG of each result handle, one after the other in one array each, and the
    edges, tests and removals per depth; the handles are freed."""
    total = sum(ds.n_vars ** 2 for ds in sets)
    adj = np.empty(total, dtype=np.uint8)
    depth = np.empty(total, dtype=np.int32)
    cpdag = np.empty(total, dtype=np.int8)
    tests = np.zeros((len(sets), MAX_DEPTHS, 3), dtype=np.int64)
    st, nd, at = (bns._lib.bns_depth_stats * MAX_DEPTHS)(), ctypes.c_int32(), 0
    for k, (h, ds) in enumerate(zip(handles, sets)):
        _ok(L.bns_skeleton_adjacency(h, _ptr(adj[at:])))
        _ok(L.bns_skeleton_removals(h, _ptr(depth[at:]), None, None, 0, None))
        _ok(L.bns_skeleton_orient(h, _ptr(cpdag[at:])))
        _ok(L.bns_skeleton_stats(h, st, MAX_DEPTHS, ctypes.byref(nd)))
        for d in range(min(nd.value, MAX_DEPTHS)):
            tests[k, d] = st[d].edges, st[d].tests_required, st[d].removed
        bns.free_skeleton(h)
        at += ds.n_vars ** 2
    return adj, depth, cpdag, tests


def run(state):
    case, L = state["case"], bns.load()
    kind = case["kind"]
    if kind == "host":
        sk = bns.bns_pc_skeleton(state["data"], state["cards"], case["alpha"], case["max_depth"], orient=True)
        sets = np.full((case["n"], case["n"], MAX_DEPTHS), -1, dtype=np.int16)
        for (i, j), members in sk.sepsets.items():
            if members:
                sets[i, j, :len(members)] = members
        return sk.adj, sk.depth, sk.cpdag, sets
    if kind == "search":
        sets = state["sets"]
        if len(sets) == 1:
            hs = [bns.skeleton_handle(sets[0], state["alphas"][0], state["depths"][0], state["opt"])]
        else:
            hs = bns.skeleton_batch_handles(sets, state["alphas"], state["depths"], state["opt"])
        return _skeletons(L, hs, sets)
    ds, opt = state["ds"], ctypes.byref(state["opt"])
    if kind == "pairs":
        stat, df, p, flags = _statistics(case["n"] * (case["n"] - 1) // 2)
        _ok(L.bns_ci_pairs(ds.handle, 0.05, opt, _ptr(stat), _ptr(df), _ptr(p), _ptr(flags)))
        return stat, df, p, flags & bns.BNS_CI_INDEPENDENT
    stat, df, p, flags = _statistics(case["tests"])
    args = (ds.handle, _ptr(state["rec"]), case["tests"], _ptr(state["pool"]), state["pool_len"], 0.05, opt,
            _ptr(stat), _ptr(df), _ptr(p), _ptr(flags))
    _ok(L.bns_ci_batch_noalloc(*args) if case["noalloc"] else L.bns_ci_batch(*args, None, None))
    return stat, df, p, flags & bns.BNS_CI_INDEPENDENT


def work(case):
    """Each column read once and the results written once; a column step per
    sample and variable of each test that any search or batch has to run (for
    a search: its depth-0 tests, the only ones known beforehand)."""
    n, m = case["n"], case["m"]
    pairs = n * (n - 1) / 2
    if case["kind"] == "ci":
        cols = 2 + (case["nz_max"] if case["tests"] == 1 else case["nz_max"] / 2)
        return dict(bytes=min(n, case["tests"] * cols) * m + 28 * case["tests"], flops=case["tests"] * cols * m)
    if case["kind"] == "pairs":
        return dict(bytes=n * m + 28 * pairs, flops=2 * pairs * m)
    if case["kind"] == "host":
        return dict(bytes=n * m + 14 * n * n, flops=2 * pairs * m)
    sizes = _sizes(case)
    return dict(bytes=sum(n * m + 6 * n * n for n, m in sizes), flops=sum(n * (n - 1) * m for n, m in sizes))


# ---------------------------------------------------------------------------
# The same in 64 bits with torch
# ---------------------------------------------------------------------------
def _statistic(N, x2, adjusted, df):
    """N: counts [..., z, y, x] in float64, df: declared; the statistic, its df and its p."""
    nx, ny, nz = N.sum(-2, keepdim=True), N.sum(-1, keepdim=True), N.sum((-1, -2), keepdim=True)
    E = nx * ny / nz.clamp(min=1)
    if x2:
        s = torch.where(E > 0, (N - E) ** 2 / E.clamp(min=1e-300), 0.0)
    else:
        s = torch.where(N > 0, 2 * N * torch.log(N.clamp(min=1) * nz / (nx * ny).clamp(min=1)), 0.0)
    s = s.sum((-1, -2, -3)).clamp(min=0)
    if adjusted:
        a, b = (nx > 0).sum((-1, -2)), (ny > 0).sum((-1, -2))
        df = ((a - 1) * (b - 1) * (nz > 0).squeeze(-1).squeeze(-1)).sum(-1)
    p = torch.where(df > 0, torch.special.gammaincc(df.double().clamp(min=1) / 2, s / 2), 1.0)
    return s, df, p


def exact(case, seed):
    if case["kind"] not in ("ci", "pairs"):
        return None  # graphs: whole numbers throughout
    n, m = case["n"], case["m"]
    data, cards = _sample(n, m, case["card_hi"], 1.25, seed)
    if case["kind"] == "ci":
        rec, pool, _ = _tests(case, seed)
        stat, df, p, flags = _statistics(case["tests"])
        for t, (x, y, nz, off) in enumerate(rec.tolist()):
            zs = pool[off:off + nz].tolist()
            cell, stride = torch.zeros(m, dtype=torch.int64, device="cuda"), 1
            for v in [x, y] + zs:
                cell += data[v].to(torch.int64) * stride
                stride *= int(cards[v])
            rx, ry = int(cards[x]), int(cards[y])
            N = torch.bincount(cell, minlength=stride).double().reshape(stride // (rx * ry), ry, rx)
            d = torch.tensor((rx - 1) * (ry - 1) * (stride // (rx * ry)), device="cuda")
            s, d, q = _statistic(N, case["x2"], case["adjusted"], d)
            stat[t], df[t], p[t] = float(s), int(d), float(q)
        flags[:] = p > 0.05
        return stat, df, p, flags
    r = int(max(cards))
    N = torch.zeros((n, r, n, r), dtype=torch.float64, device="cuda")
    for s0 in range(0, m, 20_000):  # one-hot columns of a slice of the samples, multiplied
        part = data[:, s0:s0 + 20_000]
        H = torch.stack([part == c for c in range(r)], 1).to(torch.float64).reshape(n * r, -1)
        N += (H @ H.T).reshape(n, r, n, r)
    i, j = torch.triu_indices(n, n, 1, device="cuda")
    T = N.permute(0, 2, 3, 1)[i, j][:, None]  # [pair, 1, y, x]
    c = torch.from_numpy(cards.astype(np.int64)).cuda()
    stat, df, p = _statistic(T, case["x2"], case["adjusted"], (c[i] - 1) * (c[j] - 1))
    flags = (p > 0.05).to(torch.int32)
    return tuple(a.cpu().numpy() for a in (stat, df, p, flags))
