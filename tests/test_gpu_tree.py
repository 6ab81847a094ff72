"""The LDS-claim kernel (tree.hip) where it can go wrong, bit-exact against the CPU oracle:
threshold codes at their steps, rows at and beyond the size that all waves share (and more of
them than the list holds), claim counts around a bitmap word, samples on both sides of the
dominator steps' LDS space, counter planes that fill up, and every workgroup size."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2302_13529_amd import graphgen as gg
from tests import helpers as H

pytestmark = pytest.mark.gpu


def check(gpu, n, row_ptr, col, prob, seeds, blocked, theta, key, label, slots=0, lt=False):
    print(f"[case] {label}: n={n} m={col.shape[0]} theta={theta} slots={slots}", flush=True)
    g = gpu.Graph(row_ptr, col, prob, model=gpu.IMIN_LT if lt else gpu.IMIN_IC)
    g.set_launch(slots, 0)
    D, st = g.decrease(seeds, blocked, theta, key)
    Do, so = orc.decrease(n, row_ptr, col, prob, seeds, blocked, theta, key,
                          **(dict(model=orc.LT) if lt else {}))
    assert np.array_equal(D, Do), (label, np.nonzero(D != Do)[0][:10])
    for k in ("samples", "reached", "edges_scanned", "live_edges"):
        assert st[k] == so[k], (label, k)
    g.set_small(0)  # no wavefront-level kernel
    D, st = g.decrease(seeds, blocked, theta, key)
    assert st["wave_samples"] == 0
    assert np.array_equal(D, Do), (label, np.nonzero(D != Do)[0][:10])
    for k in ("samples", "reached", "edges_scanned", "live_edges"):
        assert st[k] == so[k], (label, k)
    g.set_small(-1)
    spread, ss = g.spread(seeds, blocked, theta, key)
    assert ss["reached"] == so["reached"] and ss["live_edges"] == so["live_edges"]
    g.close()


def csr(n, src, dst, p):
    order = np.lexsort((dst, src))
    row_ptr = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(src, minlength=n), out=row_ptr[1:])
    return row_ptr, dst[order].astype(np.int32), p[order].astype(np.float32)


def test_thresholds_at_code_steps(gpu):
    """Thresholds 2^k - 1, 2^k, 2^k + 1 and mantissa steps: the byte test never loses an edge."""
    thr = sorted({t for k in range(0, 25) for d in (-1, 0, 1) for t in [2**k + d]} |
                 {(8 + i) << k for k in range(21) for i in range(8)} |
                 {((8 + i) << k) + 1 for k in range(20) for i in range(8)})
    thr = np.array([t for t in thr if 0 <= t <= 2**24])
    p = np.repeat(thr / 2.0**24, 40)  # exact in fp32: ceil(p * 2^24) is the threshold
    n = p.size + 1
    row_ptr, col, prob = csr(n, np.zeros(p.size, np.int64), np.arange(1, n), p)
    assert np.array_equal(np.ceil(prob.astype(np.float64) * 2**24), np.repeat(thr, 40))
    check(gpu, n, row_ptr, col, prob, [0], None, 3000, 11, "code steps")


@pytest.mark.parametrize("width, hubs", [(509, 3), (512, 3), (513, 3), (520, 300), (4099, 5)])
def test_heavy_rows(gpu, width, hubs):
    """Hubs of `width` out-edges, all reached in one level: rows on both sides of the 128 quads
    from which a row is shared, and more of them than the shared list holds."""
    rng = np.random.default_rng(width)
    n = 1 + hubs + 6000
    src = [np.zeros(hubs, np.int64)]
    dst = [np.arange(1, hubs + 1)]
    p = [np.full(hubs, 0.9)]
    for h in range(hubs):
        src.append(np.full(width, h + 1))
        dst.append(1 + rng.choice(n - 1, size=width, replace=False))
        p.append(np.full(width, 0.02))
    k = 4000
    src.append(rng.integers(1 + hubs, n, k))
    dst.append(rng.integers(1, n, k))
    p.append(np.full(k, 0.3))
    row_ptr, col, prob = csr(n, np.concatenate(src), np.concatenate(dst), np.concatenate(p))
    check(gpu, n, row_ptr, col, prob, [0], None, 150, 5, f"heavy {width}x{hubs}")


@pytest.mark.parametrize("extra", [0, 1, 31, 32, 33])
def test_claim_counts_around_a_word(gpu, extra):
    """nclaim = 32 + extra vertices of two in-edges, then some of one."""
    two, one = 32 + extra, 45
    n = 2 + two + one
    src = np.concatenate([np.zeros(two), np.ones(two), np.full(one, 2)]).astype(np.int64)
    dst = np.concatenate([2 + np.arange(two), 2 + np.arange(two), 2 + two + np.arange(one)])
    p = np.full(src.size, 0.5)
    row_ptr, col, prob = csr(n, src, dst, p)
    check(gpu, n, row_ptr, col, prob, [0, 1], None, 700, 3, f"words {extra}", slots=2)


@pytest.mark.parametrize("n, slots", [(3000, 0), (13000, 1), (30000, 3)])
def test_dense_samples_and_full_planes(gpu, n, slots):
    """Most vertices reached in every sample: dominator steps in LDS and in memory, and slots
    that run more samples than their counter planes hold."""
    rng = np.random.default_rng(n)
    src = np.concatenate([rng.integers(0, n, 3 * n), np.arange(0, n - 1, 3)])
    dst = np.concatenate([rng.integers(0, n, 3 * n), np.arange(1, n, 3)])
    row_ptr, col, prob = csr(n, src, dst, np.full(src.size, 0.6))
    blocked = np.zeros(n, np.uint8)
    blocked[rng.choice(np.arange(5, n), 40, replace=False)] = 1
    check(gpu, n, row_ptr, col, prob, [0, 1, 2], blocked, 150 if slots else 40, 9,
          f"dense {n}", slots=slots)


def test_every_workgroup_size(gpu):
    """The workgroup size follows from theta and the bitmap."""
    t = gg.tiny_plain()
    for theta in (1, 100, 600, 1100, 2100, 5000):
        check(gpu, t.n, t.row_ptr, t.col, t.prob, t.seeds, None, theta, theta, "tiny")


def lt_graph(n, seed, weight=None):
    """Random in-edges; a vertex's weights sum to at most 1 (unequal ones unless weight)."""
    rng = np.random.default_rng(seed)
    src, dst = rng.integers(0, n, 6 * n), rng.integers(0, n, 6 * n)
    w = np.full(src.size, 1.0) if weight else rng.random(src.size) ** 4
    w[rng.random(src.size) < 0.05] = 0.0
    total = np.bincount(dst, weights=w, minlength=n)
    scale = np.where(rng.random(n) < 0.5, 0.999, 0.7) / np.maximum(total, 1e-9)
    return csr(n, src, dst, w * scale[dst])


# reach ids per workgroup: 4096, 8192, 16384, 32768, 65532 at most; beyond, the other kernel
@pytest.mark.parametrize("n", [500, 4000, 4200, 8300, 17000, 33000, 64000, 67000])
def test_linear_threshold(gpu, n):
    row_ptr, col, prob = lt_graph(n, n)
    rng = np.random.default_rng(n)
    seeds = rng.choice(n, 40, replace=False).astype(np.int32)
    blocked = np.zeros(n, np.uint8)
    blocked[np.setdiff1d(rng.choice(n, 30, replace=False), seeds)] = 1
    check(gpu, n, row_ptr, col, prob, seeds, blocked, 60, 4, f"lt {n}", lt=True)
    check(gpu, n, row_ptr, col, prob, seeds, None, 150, 2**35 + 1, f"lt {n}", slots=2, lt=True)


def test_linear_threshold_deep_and_equal_weights(gpu):
    """A path of 3000 levels (deeper than the depth bins), and equal weights, whose draws fall
    on interval edges as often as any."""
    n = 3001
    e = [(i, i + 1, 1.0) for i in range(n - 1)]
    rp, c, p = H.csr_from_edges(n, e)
    check(gpu, n, rp, c, p, [0], None, 20, 1, "lt path", lt=True)
    row_ptr, col, prob = lt_graph(5000, 3, weight=True)
    check(gpu, 5000, row_ptr, col, prob, list(range(30)), None, 100, 1, "lt equal", lt=True)


def test_noalloc_marks_of_every_in_degree(gpu):
    """Blocked vertices with in-degrees around the 16 that one lane walks and the wavefront's
    64, in runs of neighbours and alone, every call's masks undone by the next."""
    import torch
    degrees = [0, 1, 15, 16, 17, 63, 64, 65, 300] * 20
    first = len(degrees)
    src, dst = [], []
    for v, d in enumerate(degrees):
        src += list(range(first, first + d))
        dst += [v] * d
    n = first + 301
    hub = n - 1
    src += [hub] * 300 + list(range(first))
    dst += list(range(first, first + 300)) + [(v + 1) % first for v in range(first)]
    src, dst = np.array(src), np.array(dst)
    row_ptr, col, prob = csr(n, src, dst, np.full(src.size, 0.04))
    g = gpu.Graph(row_ptr, col, prob)
    for label, marked in (("every one", range(first)), ("none", ()), ("one in 40", range(8, first, 40))):
        print(f"[case] {label}", flush=True)
        blocked = np.zeros(n, np.uint8)
        blocked[list(marked)] = 1
        out = torch.full((n,), -1, dtype=torch.int64, device="cuda")
        st = gpu.imin_decrease_noalloc(g.handle, n, [hub], blocked, 200, 5, out.data_ptr())
        torch.cuda.synchronize()
        Do, so = orc.decrease(n, row_ptr, col, prob, [hub], blocked, 200, 5)
        assert np.array_equal(out.cpu().numpy().view(np.uint64), Do), label
        assert st["reached"] == so["reached"] and st["live_edges"] == so["live_edges"]
    g.close()


@pytest.mark.parametrize("theta", [400, 5000])
def test_large_graphs_in_one_batch(gpu, theta):
    """Problems on a graph with more reach ids than the many-instance rule's 2^17, with fewer and
    with more hand-overs than there are wavefronts: chains of a few hundred vertices with
    shortcuts, beyond the packed kernel, on both sides of what one wavefront takes. Each problem
    equals its own call."""
    n = 140_001
    rng = np.random.default_rng(3)
    v = np.arange(n)
    src = np.concatenate([v, v])
    dst = np.concatenate([(v + 1) % n, (v + rng.integers(2, 400, n)) % n])
    p = np.concatenate([np.full(n, 0.99), np.full(n, 0.006)])
    row_ptr, col, prob = csr(n, src, dst, p)
    calls = (([5, 70_000], 1), ([99], 2), ([1000, 1001, 139_999], 3))
    gs = [gpu.Graph(row_ptr, col, prob) for _ in calls]
    for mode in (gpu.IMIN_AG, gpu.IMIN_GR):
        got = gpu.imin_greedy_batch([(g.handle, seeds, 2, theta, key)
                                     for g, (seeds, key) in zip(gs, calls)], mode, None)
        for (B, st), g, (seeds, key) in zip(got, gs, calls):
            Bo, so = g.greedy(seeds, 2, theta, key, mode)
            assert list(B) == list(Bo)
            for k in ("samples", "reached", "edges_scanned", "live_edges"):
                assert st[k] == so[k], (mode, k)
            assert st["wave_samples"] < st["samples"]
    for g in gs:
        g.close()
