"""Single calls with the workgroup kernel chosen by imin_set_workgroup, bit-exact against the CPU
oracle: the LDS-claim kernel in all its workgroup sizes, with its dominator and size steps in LDS
and in memory, and the kernel that claims in device memory, which otherwise runs only on graphs
with more than a million claims: its epochs, spill slots, reach counts and the wave-kernel policy
in front of it."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2302_13529_amd import graphgen as gg
from tests import helpers as H
from tests.test_gpu_limits import KEYS, csr, noalloc
from tests.test_gpu_parity import _sparse_wide_graph, check_decrease

pytestmark = pytest.mark.gpu


def dense(n, seed, lt=False):
    """Most vertices reached in every sample."""
    rng = np.random.default_rng(seed)
    src = np.concatenate([rng.integers(0, n, 3 * n), np.arange(0, n - 1)])
    dst = np.concatenate([rng.integers(0, n, 3 * n), np.arange(1, n)])
    p = np.full(src.size, 0.6)
    if lt:
        p = 0.99 / np.bincount(dst, minlength=n)[dst]
    return csr(n, src, dst, p)


def against_oracle(gpu, g, n, graph, seeds, blocked, theta, key, label, lt=False):
    model = dict(model=orc.LT) if lt else {}
    print(f"[case] {label}", flush=True)
    D, st = g.decrease(seeds, blocked, theta, key)
    Do, so = orc.decrease(n, *graph, seeds, blocked, theta, key, **model)
    assert np.array_equal(D, Do), (label, np.nonzero(D != Do)[0][:10])
    assert {k: st[k] for k in KEYS} == {k: so[k] for k in KEYS}, label
    _, ss = g.spread(seeds, blocked, theta, key)
    assert {k: ss[k] for k in KEYS} == {k: so[k] for k in KEYS}, label
    Dn, sn = noalloc(gpu, g, n, seeds, blocked, theta, key)
    assert np.array_equal(Dn, Do), label
    assert {k: sn[k] for k in KEYS} == {k: so[k] for k in KEYS}, label
    return st


@pytest.mark.parametrize("threads", [64, 128, 256, 512, 1024, -1])
@pytest.mark.parametrize("lt", [False, True])
def test_every_workgroup_size(gpu, threads, lt):
    """Samples of a few vertices, of 2,600 (in memory with 64 threads, in LDS with more) and of
    29,000 (in memory with every size)."""
    t = gg.tiny_plain()
    for n, graph, seeds, theta in ((t.n, (t.row_ptr, t.col, t.prob), t.seeds, 700),
                                   (3000, dense(3000, 1, lt), [0, 7], 90),
                                   (30_000, dense(30_000, 2, lt), [0, 1, 2], 12)):
        g = gpu.Graph(*graph, model=gpu.IMIN_LT if lt else gpu.IMIN_IC)
        g.set_workgroup(threads)
        blocked = np.zeros(n, np.uint8)
        blocked[[11, 12, 500]] = 1
        blocked[seeds] = 0
        for small in (0, 1):
            g.set_small(small)
            against_oracle(gpu, g, n, graph, seeds, blocked, theta, 2**33 + 5,
                           f"threads {threads} lt {lt} n {n} small {small}", lt)
        g.close()


def test_sizes_are_checked(gpu):
    t = gg.tiny_plain()
    g = gpu.Graph(t.row_ptr, t.col, t.prob)
    for bad in (-2, 1, 63, 96, 2048):
        with pytest.raises(gpu.IminError) as e:
            g.set_workgroup(bad)
        assert e.value.status == gpu.IMIN_EINVAL
    g.close()


def test_device_claims_epochs_wrap_and_spill(gpu):
    """One slot runs more samples than its epochs count, again in the spill slots, and the reach
    counts it keeps between them arrive."""
    n, rp, c, p, seeds = _sparse_wide_graph()
    g = gpu.Graph(rp, c, p)
    g.set_workgroup(-1)
    g.set_small(0)
    g.set_launch(1, 0)
    check_decrease(g, n, rp, c, p, seeds, None, 20000, 5, "one slot, epochs wrap")
    check_decrease(g, n, rp, c, p, seeds, None, 9000, 6, "one slot, second call")
    g.set_launch(3, 1)
    _, st = check_decrease(g, n, rp, c, p, seeds, None, 30000, 7, "spill slots, epochs wrap")
    assert st["spilled"] > 16382
    g.close()


def test_device_claims_automatic_policy(gpu):
    """The wave kernel takes a call's first round; it is dropped where it hands over most samples,
    else rounds with and without it are timed. The greedy run is the oracle's either way."""
    rp, c, p = H.csr_from_edges(300, [(i, i + 1, 1.0) for i in range(299)])
    g = gpu.Graph(rp, c, p)
    g.set_workgroup(-1)
    print("[case] path 300: dropped", flush=True)
    B, st = g.greedy([0], 3, 40, 0, gpu.IMIN_AG)
    Bo, _, so = orc.greedy(300, rp, c, p, [0], 3, 40, 0, 0)
    assert list(B) == list(Bo) and st["reached"] == so["reached"] and st["wave_samples"] == 0
    g.close()
    t = gg.tiny_plain()
    g = gpu.Graph(t.row_ptr, t.col, t.prob)
    g.set_workgroup(-1)
    for mode in (gpu.IMIN_AG, gpu.IMIN_GR):
        print(f"[case] tiny, mode {mode}: timed", flush=True)
        B, st = g.greedy(t.seeds[:2], 6, 600, 9, mode)
        Bo, _, so = orc.greedy(t.n, t.row_ptr, t.col, t.prob, t.seeds[:2], 6, 600, 9, mode)
        assert list(B) == list(Bo)
        assert {k: st[k] for k in KEYS} == {k: so[k] for k in KEYS}
        assert st["wave_samples"] > 0
    g.close()


@pytest.mark.parametrize("n, seeds, theta", [(3000, 3, 9000), (3000, 60, 9000), (3000, 60, 33000),
                                             (70_000, 2, 600), (150_000, 2, 600),
                                             (40_000, 2, 9000), (280_000, 2, 600)])
def test_preferred_sizes(gpu, n, seeds, theta):
    """Each workgroup size that is preferred by samples per slot, graph and seeds' out-edges: the
    counts are those of 512 threads, spread's too."""
    rng = np.random.default_rng(n + seeds)
    src = np.concatenate([np.arange(n), rng.integers(0, n, 4 * n)])
    dst = np.concatenate([(np.arange(n) + 1) % n, rng.integers(0, n, 4 * n)])
    for lt in (False, True):
        p = (0.99 if lt else 0.8) / np.bincount(dst, minlength=n)[dst]
        g = gpu.Graph(*csr(n, src, dst, p), model=gpu.IMIN_LT if lt else gpu.IMIN_IC)
        S = rng.choice(n, seeds, replace=False).astype(np.int32)
        print(f"[case] n {n} seeds {seeds} theta {theta} lt {lt}", flush=True)
        got = [g.decrease(S, None, theta, 5), g.spread(S, None, theta, 5)]
        g.set_workgroup(512)
        want = [g.decrease(S, None, theta, 5), g.spread(S, None, theta, 5)]
        assert np.array_equal(got[0][0], want[0][0]) and got[1][0] == want[1][0]
        for (_, a), (_, b) in zip(got, want):
            assert {k: a[k] for k in KEYS} == {k: b[k] for k in KEYS}
        g.close()


@pytest.mark.parametrize("n, p, seeds, theta", [(2000, 0.25, 20, 300), (2000, 0.32, 20, 1000),
                                                (4000, 0.9, 3, 300), (4000, 0.9, 3, 1000),
                                                (2000, 0.1, 6, 9000), (2000, 0.15, 12, 9000)])
def test_rounds_after_small_samples(gpu, n, p, seeds, theta):
    """A greedy run whose first round's samples are small changes its workgroup size: the rounds
    after it are the oracle's, and those of one size."""
    rng = np.random.default_rng(int(1000 * p) + theta)
    src = np.concatenate([np.arange(n), rng.integers(0, n, 2 * n)])
    dst = np.concatenate([(np.arange(n) + 1) % n, rng.integers(0, n, 2 * n)])
    graph = csr(n, src, dst, np.full(src.size, p))
    S = rng.choice(n, seeds, replace=False).astype(np.int32)
    g = gpu.Graph(*graph)
    for mode in (gpu.IMIN_AG, gpu.IMIN_GR):
        print(f"[case] n {n} p {p} theta {theta} mode {mode}", flush=True)
        g.set_workgroup(0)
        B, st = g.greedy(S, 5, theta, 3, mode)
        g.set_workgroup(512)
        B5, s5 = g.greedy(S, 5, theta, 3, mode)
        assert list(B) == list(B5) and {k: st[k] for k in KEYS} == {k: s5[k] for k in KEYS}
        if theta <= 300:
            Bo, _, so = orc.greedy(n, *graph, S, 5, theta, 3, mode)
            assert list(B) == list(Bo) and {k: st[k] for k in KEYS} == {k: so[k] for k in KEYS}
    g.close()
