"""The work that performance is measured on: calls a user's program makes through the public
entry points, over the range of graphs, sample counts and options they are used with.

Graphs are synthetic power-law graphs, as everywhere in this repository: R-MAT (0.57, 0.19,
0.19, 0.05) with relabelled vertices, and directed Chung-Lu (gamma 2.5), drawn on the GPU
from the case's seed. Edge values are weighted cascade ("wc", 1 / in-degree) or trivalency
("tr", one of 0.1, 0.01, 0.001); the linear-threshold model takes the "wc" weights, which sum
to 1 per vertex. A graph's handle is made once and kept, as a user's program does; a call's
seeds, blockers, sample count and Philox key come with the call.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2302_13529_amd import binding

# ------------------------------------------------------------------------------- the cases


def listed():
    return [
        # An interactive question about a small community (1000 vertices, 10 seeds): one
        # estimate of every candidate's decrease. Latency and launches are all of it.
        dict(name="decrease-1k", kind="decrease", graph="chunglu", n=1000, m=5000, prob="wc",
             model="ic", seeds=10, top=False, blocked=0, theta=1000),
        # The same question on a 131k-vertex social network after 20 blockers have been
        # placed: samples of about 10^4 vertices.
        dict(name="decrease-rmat17", kind="decrease", graph="rmat", n=1 << 17, m=1_000_000,
             prob="wc", model="ic", seeds=10, top=True, blocked=20, theta=10_000),
        # The largest network the benchmark uses (4M vertices, 35M edges): samples of
        # several 10^5 vertices, scratch far beyond every cache.
        dict(name="decrease-rmat22", kind="decrease", graph="rmat", n=1 << 22, m=35_000_000,
             prob="wc", model="ic", seeds=100, top=True, blocked=0, theta=5000),
        # The linear-threshold model on a 131k-vertex network.
        dict(name="decrease-lt-rmat17", kind="decrease", graph="rmat", n=1 << 17, m=1_000_000,
             prob="wc", model="lt", seeds=10, top=True, blocked=0, theta=5000),
        # The linear-threshold model on a 1M-vertex network.
        dict(name="decrease-lt-rmat20", kind="decrease", graph="rmat", n=1 << 20, m=8_000_000,
             prob="wc", model="lt", seeds=50, top=True, blocked=0, theta=1000),
        # The evaluation of a blocker set: Monte-Carlo spread, reachability alone.
        dict(name="spread-rmat17", kind="spread", graph="rmat", n=1 << 17, m=1_000_000,
             prob="wc", model="ic", seeds=10, top=True, blocked=50, theta=20_000),
        # A whole AdvancedGreedy run on the 131k-vertex network.
        dict(name="greedy-ag-rmat17", kind="greedy", graph="rmat", n=1 << 17, m=1_000_000,
             prob="wc", model="ic", seeds=10, top=True, theta=10_000, b=10, mode="ag"),
        # A whole GreedyReplace run on a graph of odd size under trivalency: small samples,
        # many short rounds, one host decision per replacement.
        dict(name="greedy-gr-40k", kind="greedy", graph="chunglu", n=40_111, m=401_003,
             prob="tr", model="ic", seeds=20, top=False, theta=2000, b=20, mode="gr"),
        # Many independent problems in one call (independent cascade, captured launches).
        dict(name="batch-ag-96", kind="batch", count=96, n_lo=1000, n_hi=100_000, prob="tr",
             model="ic", theta=2000, b=20, mode="ag", capture=True),
        # Many problems under the linear-threshold model with GreedyReplace.
        dict(name="batch-gr-lt-32", kind="batch", count=32, n_lo=1000, n_hi=50_000, prob="wc",
             model="lt", theta=2000, b=10, mode="gr", capture=False),
        # A burst of queries served on one resident 1M-vertex network.
        dict(name="serve-rmat20", kind="serve", graph="rmat", n=1 << 20, m=8_000_000,
             prob="wc", model="ic", queries=48, b_lo=5, b_hi=20, theta_hi=10_000),
        # The estimate into a caller's device buffer with no allocation (serving loops).
        dict(name="noalloc-rmat15", kind="noalloc", graph="rmat", n=1 << 15, m=250_000,
             prob="wc", model="ic", seeds=10, top=True, blocked=10, theta=2000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["decrease", "decrease", "spread", "greedy", "greedy", "batch", "serve",
                       "noalloc"])
    model = rng.choice(["ic", "ic", "lt"])
    prob = "wc" if model == "lt" else rng.choice(["wc", "tr"])
    if kind == "batch":
        # captured launches are an option of AdvancedGreedy batches
        mode = rng.choice(["ag", "ag", "gr"])
        return dict(kind=kind, count=_log_int(rng, 8, 96), n_lo=1000,
                    n_hi=_log_int(rng, 5000, 100_000), prob=prob, model=model,
                    theta=_log_int(rng, 500, 2000), b=rng.randint(3, 20), mode=mode,
                    capture=mode == "ag" and rng.random() < 0.5)
    # The graph; large ones only with the shapes whose samples stay affordable.
    n = _log_int(rng, 1000, 1 << (17 if kind == "noalloc" else 20))
    m = int(n * rng.uniform(4.0, 10.0))
    graph = "chunglu"
    if rng.random() < 0.5:
        n = 1 << max(10, int(round(math.log2(n))))
        graph = "rmat"
        m = int(n * rng.uniform(4.0, 9.0))
    base = dict(kind=kind, graph=graph, n=n, m=m, prob=prob, model=model)
    if kind == "serve":
        return dict(base, queries=_log_int(rng, 8, 48), b_lo=3, b_hi=rng.randint(5, 20),
                    theta_hi=_log_int(rng, 1000, 10_000))
    # samples times vertices (times rounds) at most those of the listed runs
    most = 1.3e10 if model == "ic" else 1.0e9
    theta = min(_log_int(rng, 500, 20_000 if kind == "spread" else 10_000), int(most / n))
    base.update(seeds=_log_int(rng, 1, 100), top=rng.random() < 0.5, theta=max(theta, 100))
    if kind == "greedy":
        rounds = max(1, min(rng.randint(2, 20), int(most / (n * base["theta"]))))
        return dict(base, b=rounds, mode=rng.choice(["ag", "gr"]))
    return dict(base, blocked=rng.choice([0, rng.randint(1, 50)]))


# ------------------------------------------------------------------------------ the inputs


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & (2**62 - 1))
    return g


def _csr(n, src, dst):
    key = torch.unique(src * n + dst)
    key = key[(key // n) != (key % n)]
    return key


def _rmat_keys(n, m, gen):
    """m distinct non-loop pairs (fewer when the graph has no room for them)."""
    scale = n.bit_length() - 1
    a, ab, abc = 0.57, 0.76, 0.95
    keys = torch.zeros(0, dtype=torch.int64, device="cuda")
    for _ in range(20):
        count = int((m - keys.numel()) * 1.2) + 1024
        src = torch.zeros(count, dtype=torch.int64, device="cuda")
        dst = torch.zeros(count, dtype=torch.int64, device="cuda")
        for _level in range(scale):
            r = torch.rand(count, generator=gen, device="cuda")
            src = src * 2 + (r >= ab).long()
            dst = dst * 2 + (((r >= a) & (r < ab)) | (r >= abc)).long()
        keys = torch.unique(torch.cat([keys, _csr(n, src, dst)]))
        if keys.numel() >= m:
            keep = torch.randperm(keys.numel(), generator=gen, device="cuda")[:m]
            keys = keys[keep]
            break
    perm = torch.randperm(n, generator=gen, device="cuda")
    return _csr(n, perm[keys // n], perm[keys % n])


def _chung_lu_keys(n, m, gen):
    w = torch.arange(1, n + 1, dtype=torch.float64, device="cuda") ** (-1.0 / 1.5)
    ends = []
    for _ in range(2):
        cdf = torch.cumsum(w[torch.randperm(n, generator=gen, device="cuda")], 0)
        u = torch.rand(m, generator=gen, device="cuda", dtype=torch.float64) * cdf[-1]
        ends.append(torch.searchsorted(cdf, u).clamp_(max=n - 1))
    return _csr(n, ends[0], ends[1])


def _arrays(kind, n, m, prob, gen):
    """CSR arrays on the host: row_ptr, col (int32) and edge values (float32)."""
    keys = (_rmat_keys if kind == "rmat" else _chung_lu_keys)(n, m, gen)
    src, col = keys // n, keys % n
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    if prob == "wc":
        indeg = torch.bincount(col, minlength=n).float()
        val = 1.0 / indeg[col]
    else:
        pick = torch.randint(0, 3, (col.numel(),), generator=gen, device="cuda")
        val = torch.tensor([0.1, 0.01, 0.001], device="cuda")[pick]
    return (row_ptr.int().cpu().numpy(), col.int().cpu().numpy(), val.float().cpu().numpy())


def _seeds_and_blocked(row_ptr, k, top, nblocked, rng):
    """k seeds (the largest out-degrees, or uniform) and the OutDegree blockers beside them."""
    n = row_ptr.shape[0] - 1
    k = min(k, n)
    order = np.argsort(-np.diff(row_ptr), kind="stable")
    seeds = order[:k] if top else rng.choice(n, size=k, replace=False)
    seeds = np.sort(seeds).astype(np.int32)
    blocked = None
    if nblocked:
        blocked = np.zeros(n, dtype=np.uint8)
        blocked[order[~np.isin(order, seeds)][:nblocked]] = 1
    return seeds, blocked


def _inputs(case, seed):
    arrays = _arrays(case["graph"], case["n"], case["m"], case["prob"], _gen(seed))
    rng = np.random.default_rng([int(seed) & 0xFFFFFFFF, 7])
    seeds, blocked = _seeds_and_blocked(arrays[0], case.get("seeds", 1), case.get("top", False),
                                        case.get("blocked", 0), rng)
    return arrays, seeds, blocked, rng


def _key(seed):
    return (int(seed) * 0x9E3779B97F4A7C15 + 12345) & (2**64 - 1)


def _model(case):
    return binding.IMIN_LT if case["model"] == "lt" else binding.IMIN_IC


def _mode(case):
    return binding.IMIN_GR if case["mode"] == "gr" else binding.IMIN_AG


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=dict(case), kind=kind, key=_key(seed))
    if kind == "batch":
        rng = np.random.default_rng([int(seed) & 0xFFFFFFFF, 11])
        gen = _gen(seed)
        graphs, problems = [], []
        for i in range(case["count"]):
            n = int(round(math.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
            arrays = _arrays("chunglu", n, int(n * rng.uniform(4.0, 16.0)), case["prob"], gen)
            g = binding.Graph(*arrays, model=_model(case))
            seeds, _ = _seeds_and_blocked(arrays[0], int(rng.integers(1, 51)), False, 0, rng)
            graphs.append(g)
            problems.append((g.handle, seeds, case["b"], case["theta"], st["key"] + i))
        st.update(graphs=graphs, problems=problems, mode=_mode(case),
                  launch={"graph": 1} if case["capture"] else None)
        return st
    arrays, seeds, blocked, rng = _inputs(case, seed)
    g = binding.Graph(*arrays, model=_model(case))
    st.update(graph=g, seeds=seeds, blocked=blocked)
    if kind == "serve":
        qs = []
        for i in range(case["queries"]):
            k = int(round(math.exp(rng.uniform(0.0, math.log(100.0)))))
            s, _ = _seeds_and_blocked(arrays[0], k, False, 0, rng)
            theta = int(case["theta_hi"] * rng.choice([0.1, 0.5, 1.0]))
            qs.append((s, int(rng.integers(case["b_lo"], case["b_hi"] + 1)), theta,
                       st["key"] + i))
        st.update(queries=qs, server=binding.Server(g, hbm_budget=4 << 30, max_active=64,
                                                    max_theta=case["theta_hi"]))
    elif kind == "noalloc":
        st["counts"] = torch.zeros(g.n, dtype=torch.int64, device="cuda")
    return st


# -------------------------------------------------------------------------------- one pass


def _counters(stats):
    return [stats[k] for k in ("samples", "reached", "edges_scanned", "live_edges")]


def _slots(blockers, width):
    """One row of blocker slots per problem, -1 where a run ended with fewer."""
    out = np.full((len(blockers), width), -1, dtype=np.int32)
    for row, b in zip(out, blockers):
        row[: b.shape[0]] = b
    return out


def run(state):
    case, kind = state["case"], state["kind"]
    if kind == "decrease":
        D, stats = state["graph"].decrease(state["seeds"], state["blocked"], case["theta"],
                                           state["key"])
        return dict(D=D.view(np.int64), counters=_counters(stats))
    if kind == "spread":
        spread, stats = state["graph"].spread(state["seeds"], state["blocked"], case["theta"],
                                              state["key"])
        return dict(spread=spread, counters=_counters(stats))
    if kind == "greedy":
        B, stats = state["graph"].greedy(state["seeds"], case["b"], case["theta"], state["key"],
                                         _mode(case))
        return dict(blockers=_slots([B], case["b"]), counters=_counters(stats))
    if kind == "noalloc":
        g = state["graph"]
        stats = binding.imin_decrease_noalloc(g.handle, g.n, state["seeds"], state["blocked"],
                                              case["theta"], state["key"],
                                              state["counts"].data_ptr())
        return dict(D=state["counts"], counters=_counters(stats))
    if kind == "batch":
        got = binding.imin_greedy_batch(state["problems"], state["mode"], state["launch"])
    else:
        srv = state["server"]
        tickets = [srv.submit(*q) for q in state["queries"]]
        while srv.step() != (0, 0):
            pass
        srv.completed()
        got = [srv.result(t, q[1]) for t, q in zip(tickets, state["queries"])]
    return dict(sizes=np.array([b.shape[0] for b, _ in got], dtype=np.int64),
                blockers=_slots([b for b, _ in got], case.get("b", case.get("b_hi"))),
                counters=np.array([_counters(s) for _, s in got], dtype=np.int64))


# ------------------------------------------------------------------- work and exact results


def work(case):
    """Each input read once, each output written once; operations: the coins of the seeds'
    own out-edges (the least that every sample draws), one Philox4x32-10 block (10 rounds of
    8 integer operations) per 4 edges."""
    if case["kind"] == "batch":
        lo, hi = case["n_lo"], case["n_hi"]
        n = case["count"] * ((hi - lo) / math.log(hi / lo) if hi > lo else lo)
        m, samples, edges = 10 * n, case["count"] * case["theta"] * case["b"], 25 * 10
        out = case["count"] * (4 * case["b"] + 32)
    else:
        n, m = case["n"], case["m"]
        if case["kind"] == "serve":
            samples = case["queries"] * case["theta_hi"] * 0.53 * (case["b_lo"] + case["b_hi"]) / 2
            edges = 21.5 * m / n
            out = case["queries"] * (2 * (case["b_lo"] + case["b_hi"]) + 32)
        else:
            samples = case["theta"] * case.get("b", 1)
            edges = case["seeds"] * m / n
            out = {"decrease": 8 * n, "noalloc": 8 * n, "spread": 40}.get(
                case["kind"], 4 * case.get("b", 0) + 32)
    return dict(bytes=8.0 * m + 4.0 * n + out, flops=20.0 * samples * edges)


def _philox(c0, c1, key, device):
    """Philox4x32-10 at counters (c0, c1, 0, 0), int64 tensors holding 32-bit words."""
    M = 0xFFFFFFFF
    k0, k1 = key & M, key >> 32
    x0, x1 = torch.broadcast_tensors(c0, c1)
    x2 = torch.zeros((), dtype=torch.int64, device=device)
    x3 = torch.zeros((), dtype=torch.int64, device=device)

    def mul(a, b):  # 32 x 32 -> (high, low), within signed 64 bits
        lo = (a & 0xFFFF) * b
        hi = (a >> 16) * b
        s = lo + ((hi & 0xFFFF) << 16)
        return (hi >> 16) + (s >> 32), s & M

    for _ in range(10):
        h0, l0 = mul(x0, 0xD2511F53)
        h1, l1 = mul(x2, 0xCD9E8D57)
        x0, x1, x2, x3 = h1 ^ x1 ^ k0, l1, h0 ^ x3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return x0, x1, x2, x3


def _live(thr, j, key):
    """Live edges [m, samples j] under the independent cascade: coin < ceil(p * 2^24)."""
    m, dev = thr.numel(), thr.device
    quads = torch.arange((m + 3) // 4, device=dev).unsqueeze(1)
    w = torch.stack(_philox(quads, j.unsqueeze(0), key, dev), 1).reshape(-1, j.numel())
    return (w[:m] >> 8) < thr.unsqueeze(1)


def _idom_counts(n, out, roots):
    """Subtree sizes in the dominator tree of one sample: out[u] lists the live targets."""
    order, parent, seen, preds = [], {}, set(roots), {}
    level = list(roots)
    index = {}
    while level:
        nxt = []
        for u in level:
            for v in out.get(u, ()):
                if v in roots:
                    continue
                if v not in seen:
                    seen.add(v)
                    parent[v] = -1 if u in roots else u
                    index[v] = len(order)
                    order.append(v)
                    nxt.append(v)
                preds.setdefault(v, []).append(-1 if u in roots else u)
        level = nxt
    index[-1] = -1
    idom = dict(parent)
    idom[-1] = -1
    changed = True
    while changed:
        changed = False
        for v in order:
            x = idom[v]
            for y in preds[v]:
                while x != y:
                    if index[x] > index[y]:
                        x = idom[x]
                    else:
                        y = idom[y]
            if x != idom[v]:
                idom[v] = x
                changed = True
    # a dominator comes before what it dominates in breadth-first order
    size = {v: 1 for v in order}
    for v in reversed(order):
        if idom[v] != -1:
            size[idom[v]] += size[v]
    return size


def exact(case, seed):
    if case["model"] != "ic":
        return None
    if case["kind"] == "spread" and case["m"] * case["theta"] <= 2.1e10:
        return _exact_spread(case, seed)
    if case["kind"] == "decrease" and case["m"] * case["theta"] <= 2e7:
        return _exact_decrease(case, seed)
    return None


def _problem(case, seed):
    (row_ptr, col, val), seeds, blocked, _ = _inputs(case, seed)
    dev = torch.device("cuda")
    row_ptr = torch.from_numpy(row_ptr).to(dev).long()
    col = torch.from_numpy(col).to(dev).long()
    src = torch.repeat_interleave(torch.arange(case["n"], device=dev), row_ptr.diff())
    thr = torch.ceil(torch.from_numpy(val).to(dev).double() * 2.0**24).long()
    is_seed = torch.zeros(case["n"], dtype=torch.bool, device=dev)
    is_seed[torch.from_numpy(seeds).to(dev).long()] = True
    closed = is_seed.clone()
    if blocked is not None:
        closed |= torch.from_numpy(blocked).to(dev).bool()
    thr[closed[col]] = 0  # an edge into a seed or a blocked vertex is never live
    return src, col, thr, is_seed, row_ptr.diff()


def _exact_spread(case, seed):
    src, col, thr, is_seed, deg = _problem(case, seed)
    dev, theta, n = src.device, case["theta"], case["n"]
    first = torch.cumsum(deg, 0) - deg
    roots = is_seed.nonzero().flatten()
    step = max(16, min(512, int(2e8 / max(case["m"], n))))
    reached = scanned = lives = 0
    for j0 in range(0, theta, step):
        k = min(theta, j0 + step) - j0  # samples of this chunk
        live = _live(thr, torch.arange(j0, j0 + k, device=dev), _key(seed))
        seen = torch.zeros(n * k, dtype=torch.bool, device=dev)
        # the frontier as (vertex, sample) pairs
        v = roots.repeat_interleave(k)
        j = torch.arange(k, device=dev).repeat(roots.numel())
        while v.numel():
            d = deg[v]
            at = torch.repeat_interleave(torch.arange(v.numel(), device=dev), d)
            e = first[v][at] + torch.arange(at.numel(), device=dev) - (torch.cumsum(d, 0) - d)[at]
            jj = j[at]
            on = live[e, jj]
            key = col[e[on]] * k + jj[on]
            scanned += at.numel()
            lives += key.numel()
            key = torch.unique(key[~seen[key]])
            seen[key] = True
            reached += key.numel()
            v, j = key // k, key % k
    return dict(spread=float(roots.numel()) + reached / theta,
                counters=[theta, reached, scanned, lives])


def _exact_decrease(case, seed):
    src, col, thr, is_seed, deg = _problem(case, seed)
    theta, n = case["theta"], case["n"]
    live = _live(thr, torch.arange(theta, device=src.device), _key(seed)).cpu().numpy()
    src, col, deg = src.cpu().numpy(), col.cpu().numpy(), deg.cpu().numpy()
    roots = [int(v) for v in is_seed.nonzero().flatten().cpu()]
    rset = set(roots)
    D = np.zeros(n, dtype=np.int64)
    reached = scanned = lives = 0
    base = int(deg[roots].sum())
    for j in range(theta):
        out = {}
        for e in np.flatnonzero(live[:, j]):
            out.setdefault(int(src[e]), []).append(int(col[e]))
        size = _idom_counts(n, out, rset)
        for v, c in size.items():
            D[v] += c
        reached += len(size)
        scanned += base + sum(int(deg[v]) for v in size)
        lives += sum(len(out.get(v, ())) for v in size) + sum(len(out.get(v, ())) for v in roots)
    return dict(D=D, counters=[theta, reached, scanned, lives])
