"""What a call accepts and what its scratch holds, where the kernels' own sizes could narrow it:
extra edges that a quarter of the vertices covers, though a quarter of the reachable ones does
not, and graphs of many edges through the no-allocation call."""
import numpy as np
import pytest

from oracle import oracle as orc

pytestmark = pytest.mark.gpu

KEYS = ("samples", "reached", "edges_scanned", "live_edges")


def csr(n, src, dst, p):
    order = np.lexsort((dst, src))
    row_ptr = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(src, minlength=n), out=row_ptr[1:])
    return row_ptr, dst[order].astype(np.int32), p[order].astype(np.float32)


def core_graph(n, core, extra, seed):
    """Vertices 0..core-1 hang from vertex 0 in a random tree of edges that are always live, with
    `extra` more such edges among them; the other vertices have no edges."""
    rng = np.random.default_rng(seed)
    child = np.arange(1, core)
    src = np.concatenate([(child * rng.random(core - 1)).astype(np.int64),
                          rng.integers(1, core, extra)])
    dst = np.concatenate([child, rng.integers(1, core, extra)])
    return csr(n, src, dst, np.ones(src.size))


def noalloc(gpu, g, n, seeds, blocked, theta, key):
    import torch
    out = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    st = gpu.imin_decrease_noalloc(g.handle, n, seeds, blocked, theta, key, out.data_ptr())
    torch.cuda.synchronize()
    return out.cpu().numpy().view(np.uint64), st


def test_extra_edges_of_a_quarter_of_the_vertices_do_not_spill(gpu):
    """17,000 extra edges a sample: more than a quarter of the 6,000 reachable vertices (and than
    the least capacity, 4,096), fewer than a quarter of the 80,000 there are."""
    n, theta = 80_000, 20
    row_ptr, col, prob = core_graph(n, 6000, 17_000, 1)
    Do, so = orc.decrease(n, row_ptr, col, prob, [0], None, theta, 3)
    g = gpu.Graph(row_ptr, col, prob)
    print("[case] extra edges, decrease", flush=True)
    D, st = g.decrease([0], None, theta, 3)
    assert np.array_equal(D, Do) and st["spilled"] == 0
    print("[case] extra edges, noalloc", flush=True)
    D, st = noalloc(gpu, g, n, [0], None, theta, 3)
    assert np.array_equal(D, Do) and st["spilled"] == 0
    assert {k: st[k] for k in KEYS} == {k: so[k] for k in KEYS}
    g.close()


def test_extra_edges_in_a_batch_do_not_spill(gpu):
    """The same for a batch on a graph of more than 2^17 reach ids."""
    n, theta = 500_000, 6
    row_ptr, col, prob = core_graph(n, 140_000, 90_000, 2)
    g, h = gpu.Graph(row_ptr, col, prob), gpu.Graph(row_ptr, col, prob)
    print("[case] extra edges, batch", flush=True)
    got = gpu.imin_greedy_batch([(g.handle, [0], 1, theta, 3), (h.handle, [0], 1, theta, 4)])
    for (B, st), key in zip(got, (3, 4)):
        Bo, so = g.greedy([0], 1, theta, key, gpu.IMIN_AG)
        assert list(B) == list(Bo) and st["spilled"] == 0 == so["spilled"]
        assert {k: st[k] for k in KEYS} == {k: so[k] for k in KEYS}
    g.close()
    h.close()


@pytest.mark.parametrize("n, m", [(1 << 18, 8_000_000), (200_000, 10_000_000)])
def test_noalloc_takes_graphs_of_many_edges(gpu, n, m):
    """A large slot of all m extra edges takes 16 m bytes, of which one fits the array beside the
    ordinary slots and two do not."""
    rng = np.random.default_rng(n)
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    row_ptr, col, prob = csr(n, src, dst, 1.0 / np.bincount(dst, minlength=n)[dst])
    g = gpu.Graph(row_ptr, col, prob)
    seeds = np.arange(40, dtype=np.int32)
    print(f"[case] n={n} m={m}", flush=True)
    D, st = noalloc(gpu, g, n, seeds, None, 300, 3)
    assert st["wave_samples"] > 0  # few slots: the wave kernel takes the small samples
    Do, so = g.decrease(seeds, None, 300, 3)
    assert np.array_equal(D, Do)
    assert {k: st[k] for k in KEYS} == {k: so[k] for k in KEYS}
    g.close()


def test_noalloc_wave_kernel_gives_up(gpu):
    """Few slots and only large samples: every wave lists the rest of its samples untried."""
    n, theta = 300_000, 600
    row_ptr, col, prob = core_graph(n, 262_000, 1000, 5)
    g = gpu.Graph(row_ptr, col, prob)
    print("[case] gives up", flush=True)
    D, st = noalloc(gpu, g, n, [0], None, theta, 3)
    Do, so = g.decrease([0], None, theta, 3)
    assert np.array_equal(D, Do) and st["wave_samples"] == 0
    assert {k: st[k] for k in KEYS} == {k: so[k] for k in KEYS}
    g.close()


def test_many_small_samples_in_single_calls(gpu):
    """Claims that leave one slot a compute unit, and 64 samples and more for each: the wave kernel
    takes the small samples of decrease, spread and a greedy run's rounds."""
    n, m, theta = 1_000_000, 7_000_000, 17_000
    rng = np.random.default_rng(8)
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    p = 0.9 / np.bincount(dst, minlength=n)[dst]
    g = gpu.Graph(*csr(n, src, dst, p))
    seeds = [5, 77, 123_456]
    print("[case] many small samples", flush=True)
    got = g.decrease(seeds, None, theta, 3), g.spread(seeds, None, theta, 3)
    assert got[0][1]["wave_samples"] > theta // 2 and got[1][1]["wave_samples"] > theta // 2
    B, st = g.greedy(seeds, 3, theta, 3, gpu.IMIN_AG)
    assert st["wave_samples"] > theta
    g.set_small(0)
    want = g.decrease(seeds, None, theta, 3), g.spread(seeds, None, theta, 3)
    assert np.array_equal(got[0][0], want[0][0]) and got[1][0] == want[1][0]
    for (_, a), (_, b) in zip(got, want):
        assert {k: a[k] for k in KEYS} == {k: b[k] for k in KEYS} and b["wave_samples"] == 0
    Bo, so = g.greedy(seeds, 3, theta, 3, gpu.IMIN_AG)
    assert list(B) == list(Bo) and {k: st[k] for k in KEYS} == {k: so[k] for k in KEYS}
    g.close()


@pytest.mark.parametrize("lt", [False, True])
def test_spread_scratch_is_row_ranges(gpu, lt):
    """A reachability-only call keeps 12 bytes a reach id for each of at most 16 slots a compute
    unit, or 28 bytes for two; a decrease call beside it shares that space, and both are right."""
    import torch
    n = 150_000
    rng = np.random.default_rng(9)
    src = np.concatenate([np.arange(n), rng.integers(0, n, 3 * n)])
    dst = np.concatenate([(np.arange(n) + 1) % n, rng.integers(0, n, 3 * n)])
    p = 0.9 / np.bincount(dst, minlength=n)[dst]
    graph = csr(n, src, dst, p)
    g = gpu.Graph(*graph, model=gpu.IMIN_LT if lt else gpu.IMIN_IC)
    # many seeds: the smallest workgroups
    seeds = rng.choice(n, 400, replace=False).astype(np.int32)
    print(f"[case] scratch, lt {lt}", flush=True)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    s1, st = g.spread(seeds, None, 5000, 3)
    held = before - torch.cuda.mem_get_info()[0]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert held <= cus * n * max(16 * 12, 2 * 28) + (64 << 20), held
    D, sd = g.decrease(seeds, None, 5000, 3)
    s2, su = g.spread(seeds, None, 5000, 3)
    assert s1 == s2 and {k: st[k] for k in KEYS} == {k: sd[k] for k in KEYS}
    assert int(D.max()) > 0 and {k: st[k] for k in KEYS} == {k: su[k] for k in KEYS}
    D2, _ = g.decrease(seeds, None, 5000, 3)
    assert np.array_equal(D, D2)
    g.close()
    h = gpu.Graph(*graph, model=gpu.IMIN_LT if lt else gpu.IMIN_IC)
    D3, _ = h.decrease(seeds, None, 5000, 3)
    assert np.array_equal(D, D3)
    h.close()


def test_forced_wave_kernel_keeps_few_slots(gpu):
    """Ten hand-overs need no more than the 64 slots that go with the wave kernel."""
    import torch
    n = 200_000
    src, dst = np.arange(n), (np.arange(n) + 1) % n
    p = np.where(src < 300, 1.0, 0.0)
    twice = np.concatenate([src, src]), np.concatenate([dst, dst]), np.concatenate([p, 0 * p])
    g = gpu.Graph(*csr(n, *twice))
    g.set_small(1)
    print("[case] forced wave kernel", flush=True)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    D, st = g.decrease([0], None, 10, 3)
    held = before - torch.cuda.mem_get_info()[0]
    assert st["wave_samples"] == 0 and st["reached"] == 10 * 300
    assert held <= 64 * (26 * n + 16 * (n // 4)) + (64 << 20), held
    g.close()
