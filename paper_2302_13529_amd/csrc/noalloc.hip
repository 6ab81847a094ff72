// noalloc.hip -- imin_decrease_noalloc: Algorithm 2 of arXiv 2302.13529 (the same counts as
// imin_decrease) for callers that cannot allocate device memory: code under HIP graph
// capture, tight serving loops, harnesses that forbid allocation.
//
// Every scratch buffer of the call -- the seed staging, the blocked marks, the wave kernel's
// hand-over list, the workgroup kernel's slot maps, local records, level starts and extra-edge
// lists, its overflow list and the large-capacity spill slots -- is carved from one
// file-scope device array of kScratchBytes per GPU. The caller passes the graph (made
// resident by imin_graph_create), the host seed set and blocked marks, and a device buffer of
// n uint64 counts, which the kernels write directly. No hipMalloc, hipFree or other
// allocating routine is called.
#include "graph.h"

#include <algorithm>
#include <cstring>
#include <mutex>

namespace {

constexpr size_t kScratchBytes = size_t(256) << 20;  // IMIN_NOALLOC_SCRATCH_BYTES

// The scratch array. In host code this name stands for the symbol, not for a device
// address: host code only ever uses the per-device address that hipGetSymbolAddress returns.
__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned char *g_scratch_ptr[kMaxDevices] = {};

// The device address of `scratch` on the current device `dev`, looked up once per device.
int scratch_on(int dev, unsigned char **out)
{
    if (dev < 0 || dev >= kMaxDevices) return IMIN_EDEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return IMIN_EDEVICE;
        }
        g_scratch_ptr[dev] = static_cast<unsigned char *>(p);
    }
    *out = g_scratch_ptr[dev];
    return IMIN_OK;
}

constexpr int kBlock = 256;

// Distinct seeds: the first thread to set a seed's bit appends it (any order; the counts do
// not depend on the order of the seed list).
__global__ void seed_set_kernel(const int32_t *S, int32_t nS, uint32_t *bits, int32_t *out,
                                uint32_t *count)
{
    for (int32_t i = blockIdx.x * kBlock + threadIdx.x; i < nS; i += gridDim.x * kBlock) {
        const int32_t s = S[i];
        const uint32_t bit = 1u << (s & 31);
        if (!(atomicOr(&bits[s >> 5], bit) & bit)) out[atomicAdd(count, 1u)] = s;
    }
}

// In-edge thresholds of every vertex v with marks[v] != 0: 0, or restored from orig. A lane
// looks at one vertex and walks a few in-edges itself; the wavefront walks longer lists
// together. Ten marked vertices of a 32k-vertex R-MAT graph (up to 1,000 in-edges): 197 us and
// 400 us to restore with one lane for each; the call took 1.74 ms then and takes 1.10 so.
constexpr int32_t kOwnEdges = 16;

__global__ void mask_marked_kernel(uint32_t *thr, uint4 *rec, const uint32_t *orig, const int32_t *in_ptr,
                                   const int32_t *in_edge, const uint8_t *marks, int32_t n,
                                   int restore)
{
    const int lane = threadIdx.x & 63;
    auto set = [&](int32_t k) {
        const int32_t e = in_edge[k];
        const uint32_t t = restore ? orig[e] : 0u;
        thr[e] = t;
        if (rec) rec[e].w = t;
    };
    // a wavefront's 64 vertices start at v0
    for (int64_t v0 = blockIdx.x * (int64_t)kBlock + threadIdx.x - lane; v0 < n;
         v0 += (int64_t)gridDim.x * kBlock) {
        const int64_t v = v0 + lane;
        int32_t first = 0, last = 0;
        if (v < n && marks[v]) {
            first = in_ptr[v];
            last = in_ptr[v + 1];
        }
        const bool wide = last - first > kOwnEdges;
        if (!wide)
            for (int32_t k = first; k < last; ++k) set(k);
        for (unsigned long long w = __ballot(wide); w; w &= w - 1) {
            const int l = __builtin_ctzll(w);
            const int32_t end = __shfl(last, l, 64);
#pragma unroll 4
            for (int32_t k = __shfl(first, l, 64) + lane; k < end; k += 64) set(k);
        }
    }
}

int grid_of(int64_t count)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>(4096, (count + kBlock - 1) / kBlock));
}

// A bump allocator over the scratch array (offsets only; nothing is allocated).
struct Carve {
    unsigned char *base;
    size_t used = 0;
    bool fits = true;
    template <class T>
    T *take(size_t count)
    {
        const size_t off = (used + 255) & ~size_t(255);
        const size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
        if (off + bytes > kScratchBytes) {
            fits = false;
            return nullptr;
        }
        used = off + bytes;
        return reinterpret_cast<T *>(base + off);
    }
};

// The LDS-claim kernel's scratch of `slots` slots in the carve.
bool carve_tree_ws(Carve &c, imin::TreeWs &ws, int32_t slots, int64_t lcap, int64_t xcap,
                   int64_t nclaim, int64_t words)
{
    const size_t off = (c.used + 255) & ~size_t(255);
    const size_t bytes =
        imin::host::carve_tree(ws, c.base + off, slots, lcap, xcap, nclaim, words);
    if (off + bytes > kScratchBytes) return c.fits = false;
    c.used = off + bytes;
    return true;
}

// The LDS-claim kernel's scratch: every reachable vertex and the root fit a slot, and there are
// as many slots as the rest of the array holds, up to the usual count. An extra edge takes 16
// bytes here and 8 in the kernel of large claim sets, and a large slot holds all m of them: so
// there are two only where that costs no slot, and where not even one ordinary slot is left
// beside a single large one, it holds fewer extra edges. With that, what fits the other kernel's
// layout fits this one.
bool carve_tree_call(Carve &c, const imin_graph *g, uint32_t theta, imin::TreeShape &shape,
                     imin::TreeWs &main_tw, imin::TreeWs &big_tw)
{
    const bool lt = g->model == IMIN_LT;
    const int64_t cap = (int64_t)g->nreach + 1, nclaim = lt ? 0 : g->nclaim;
    const int64_t words = ((int64_t)g->nreach + 31) / 32, xmax = (int64_t)g->m + 1;
    int64_t xcap = lt ? 1 : imin::host::extra_cap(g->n, g->m);
    imin::tree_shape(imin::host::tree_fit(g, theta, false), shape);
    const int64_t full = (int64_t)shape.per_cu * g->num_cus;
    auto room = [&](int64_t x) {  // slots of x extra edges in what is left
        imin::TreeWs one;
        const size_t per = imin::host::carve_tree(one, nullptr, 1, cap, x, nclaim, words);
        const size_t used = (c.used + 255) & ~size_t(255);
        return used > kScratchBytes ? 0 : (int64_t)((kScratchBytes - used) / per);
    };
    const Carve start = c;
    for (int32_t large = lt || xcap >= xmax ? 0 : 2; large >= 0; --large) {
        c = start;
        big_tw = imin::TreeWs();
        if (large > 0 && !carve_tree_ws(c, big_tw, large, cap, xmax, nclaim, 0)) {
            if (large > 1) continue;
            return false;
        }
        if (large > 1 && room(xcap) < full) continue;
        if (large == 1)
            while (xcap > 1 && room(xcap) == 0) xcap /= 2;
        const int32_t slots = (int32_t)std::max<int64_t>(1, std::min(full, room(xcap)));
        if (slots <= g->num_cus) {  // at most one a compute unit: the largest workgroup
            imin::TreeFit fit = imin::host::tree_fit(g, theta, false);
            fit.most = slots;
            imin::tree_shape(fit, shape);
        }
        return carve_tree_ws(c, main_tw, slots, cap, xcap, nclaim, words);
    }
    return false;
}

// Slot-major workgroup-kernel scratch of `slots` slots in the carve.
bool carve_ws(Carve &c, imin::Workspace &ws, int64_t n, int32_t slots, int64_t lcap, int64_t xcap)
{
    int32_t lbits = 1;
    while (lbits < 32 && (int64_t(1) << lbits) <= lcap) ++lbits;
    if (lbits > 31) return false;
    const size_t S = (size_t)slots;
    ws.map = c.take<unsigned long long>(S * (size_t)n);
    ws.loc = c.take<imin::LocalVtx>(S * (size_t)lcap);
    ws.lvl = c.take<int32_t>(S * (size_t)(lcap + 1));
    ws.extra = c.take<int2>(S * (size_t)std::max<int64_t>(xcap, 1));
    ws.epoch = c.take<uint32_t>(S);
    ws.dirty = c.take<uint32_t>(S);
    ws.rng = c.take<int2>(S * (size_t)lcap);
    ws.slots = slots;
    ws.n = n;
    ws.lcap = lcap;
    ws.xcap = xcap;
    ws.lbits = lbits;
    return c.fits;
}

}  // namespace

using namespace imin::host;

extern "C" {

int imin_decrease_noalloc(imin_graph *g, const int32_t *S, int32_t nS, const uint8_t *blocked,
                          uint32_t theta, uint64_t seed, uint64_t *d_counts, imin_stats *stats)
{
    if (!g || !S || nS <= 0 || theta == 0 || !d_counts) return IMIN_EINVAL;
    if (theta > kMaxTheta) return IMIN_ERANGE;
    for (int32_t i = 0; i < nS; ++i) {
        if (S[i] < 0 || S[i] >= g->n) return IMIN_EINVAL;
        if (blocked && blocked[S[i]]) return IMIN_EINVAL;  // B is a subset of V \ S
    }
    g->seed_edges = out_edges(g, S, (size_t)nS);
    g->prefer = 0;
    if (!ok(hipSetDevice(g->device))) return IMIN_EDEVICE;
    unsigned char *base = nullptr;
    int rc = scratch_on(g->device, &base);
    if (rc) return rc;

    // Layout of this call's scratch.
    const int64_t n = g->n, m = g->m;
    const int64_t lcap = n + 1, xmax = m + 1;
    const int64_t xcap = extra_cap(n, m);
    Carve c{base};
    uint32_t *bits = c.take<uint32_t>((size_t)g->words);
    int32_t *s_in = c.take<int32_t>((size_t)nS);
    int32_t *s_set = c.take<int32_t>((size_t)nS);
    uint32_t *s_count = c.take<uint32_t>(1);
    uint8_t *marks = blocked ? c.take<uint8_t>((size_t)n) : nullptr;
    uint32_t *sj = c.take<uint32_t>(theta);
    uint32_t *ovf = c.take<uint32_t>(theta);
    imin::Workspace main_ws, big_ws;
    imin::TreeWs main_tw, big_tw;
    const bool tree = tree_on(g);
    if (tree) {
        if (!c.fits || !carve_tree_call(c, g, theta, g->shape, main_tw, big_tw)) return IMIN_ERANGE;
    } else {
        if (xcap < xmax && !carve_ws(c, big_ws, n, 2, lcap, xmax)) return IMIN_ERANGE;
        if (!c.fits) return IMIN_ERANGE;
        const size_t fixed = c.used;
        // as many workgroup slots as the rest holds, up to the usual count
        Carve probe{base, fixed};
        imin::Workspace one;
        if (!carve_ws(probe, one, n, 1, lcap, xcap)) return IMIN_ERANGE;
        const size_t per_slot = probe.used - fixed + 7 * 256;
        const int32_t slots = (int32_t)std::max<size_t>(
            1, std::min<size_t>((size_t)imin::kSlotsPerCu * g->num_cus,
                                (kScratchBytes - fixed) / per_slot));
        if (!carve_ws(c, main_ws, n, slots, lcap, xcap)) return IMIN_ERANGE;
        if (xcap >= xmax) big_ws = imin::Workspace();
    }

    hipStream_t st = g->stream;
    uint32_t *thr = reinterpret_cast<uint32_t *>(g->d_thr4);
    const uint32_t *orig = reinterpret_cast<const uint32_t *>(g->d_thr_orig);
    // Thresholds: undo what an earlier call on this graph left masked; from here until the
    // end of the call the graph's masking state is unknown to the other entry points.
    if (!g->mask_known) {
        const int64_t quads = std::max<int64_t>((m + 3) / 4, 1);
        if (!ok(hipMemcpyAsync(g->d_thr4, g->d_thr_orig, (size_t)quads * sizeof(uint4),
                               hipMemcpyDeviceToDevice, st)) ||
            (g->mask_rec() && !ok(imin::launch_edge_restore(orig, m, g->mask_rec(), st))))
            return IMIN_EDEVICE;
    } else if (!g->masked.empty()) {
        if (!ok(hipMemcpyAsync(g->d_list, g->masked.data(), g->masked.size() * sizeof(int32_t),
                               hipMemcpyHostToDevice, st)) ||
            !ok(imin::launch_mask_list(thr, g->mask_rec(), orig, g->d_in_ptr, g->d_in_edge, g->d_list,
                                       (int32_t)g->masked.size(), 1, st)))
            return IMIN_EDEVICE;
    }
    g->masked.clear();
    g->mask_known = false;

    // Distinct seeds, blocked marks, cleared counters and slot maps.
    uint32_t nseeds = 0;
    if (!ok(imin::launch_fill_u32(bits, g->words, 0u, st)) ||
        !ok(imin::launch_fill_u32(s_count, 1, 0u, st)) ||
        !ok(hipMemcpyAsync(s_in, S, (size_t)nS * sizeof(int32_t), hipMemcpyHostToDevice, st)) ||
        (blocked && !ok(hipMemcpyAsync(marks, blocked, (size_t)n, hipMemcpyHostToDevice, st))))
        return IMIN_EDEVICE;
    hipLaunchKernelGGL(seed_set_kernel, dim3(grid_of(nS)), dim3(kBlock), 0, st, s_in, nS, bits,
                       s_set, s_count);
    if (!ok(hipGetLastError()) ||
        !ok(hipMemcpyAsync(&nseeds, s_count, sizeof(nseeds), hipMemcpyDeviceToHost, st)) ||
        !ok(hipStreamSynchronize(st)))
        return IMIN_EDEVICE;
    if (!ok(imin::launch_mask_list(thr, g->mask_rec(), orig, g->d_in_ptr, g->d_in_edge, s_set, (int32_t)nseeds,
                                   0, st)))
        return IMIN_EDEVICE;
    if (blocked) {
        hipLaunchKernelGGL(mask_marked_kernel, dim3(grid_of(n)), dim3(kBlock), 0, st, thr, g->mask_rec(), orig,
                           g->d_in_ptr, g->d_in_edge, marks, (int32_t)n, 0);
        if (!ok(hipGetLastError())) return IMIN_EDEVICE;
    }
    const imin::Workspace *wss[2] = {&main_ws, &big_ws};
    for (const imin::Workspace *w : wss) {
        if (w->slots <= 0) continue;
        if (!ok(imin::launch_fill_u32(reinterpret_cast<uint32_t *>(w->map),
                                      2 * (int64_t)w->slots * w->n, 0u, st)) ||
            !ok(imin::launch_fill_u32(w->epoch, w->slots, 0u, st)) ||
            !ok(imin::launch_fill_u32(w->dirty, w->slots, 0u, st)))
            return IMIN_EDEVICE;
    }
    if (tree && (!ok(imin::launch_fill_u32(main_tw.planes,
                                              (int64_t)main_tw.slots * imin::kTreePlanes *
                                                  main_tw.words, 0u, st)) ||
                    !ok(imin::launch_fill_u64(g->d_D + n, g->nreach, 0ull, st))))
        return IMIN_EDEVICE;
    if (!ok(imin::launch_fill_u64(reinterpret_cast<unsigned long long *>(d_counts), n, 0ull, st)) ||
        !ok(imin::launch_fill_u64(g->d_stats, kStats, 0ull, st)) ||
        !ok(imin::launch_fill_u32(g->d_ctrl, imin::kCtrlWords, 0u, st)) ||
        !ok(imin::launch_fill_u32(g->d_sctrl, 2, 0u, st)))
        return IMIN_EDEVICE;

    // The graph as the one instance of the wave kernel, counting into the caller's buffer.
    imin::InstanceDesc I{};
    I.row_ptr = g->d_row_ptr;
    I.col4 = g->d_col4;
    I.edge = g->d_edge;
    I.thr4 = g->d_thr4;
    I.lo4 = g->d_lo4;
    I.tl = g->d_tl;
    I.in_ptr = g->d_in_ptr;
    I.in_edge = g->d_in_edge;
    I.inelig = bits;
    I.seeds = s_set;
    I.D = reinterpret_cast<unsigned long long *>(d_counts);
    I.stats = g->d_stats;
    I.thr_orig = g->d_thr_orig;
    I.ctrl = g->d_ctrl;
    I.nseeds = (int32_t)nseeds;
    I.n = g->n;
    I.nquads = (int32_t)std::max<int64_t>((m + 3) / 4, 1);
    I.nclaim = g->nclaim;
    I.nreach = g->nreach;
    I.tedge = g->d_tedge;
    I.code = g->d_code;
    I.rid_vtx = g->d_rid_vtx;
    I.seed_lo = (uint32_t)seed;
    I.seed_hi = (uint32_t)(seed >> 32);
    I.theta = theta;
    I.sample_base = 0;
    if (!ok(hipEventRecord(g->ev0, st)) ||
        !ok(hipMemcpyAsync(g->d_inst, &I, sizeof(I), hipMemcpyHostToDevice, st)))
        return IMIN_EDEVICE;
    // The LDS-claim kernel takes every sample itself, unless there are very many, or 16 and more a
    // slot (32 where the seeds have hardly any out-edges) on graphs whose slots in the array are
    // fewer than the compute units, where the wave kernel alone fills the chip. 10,000 samples of a
    // 131k-vertex trivalency graph, 67 slots, 1.80 ms without it and 0.37 with it; 2,000 from one
    // seed of a 524k-vertex graph, 9 slots, 2.33 and 0.54; but 2,000 from one of a 131k-vertex R-MAT
    // graph, some 90 slots, 0.56 and 0.65, and 500 0.18 and 0.30. The kernel of large claim sets
    // takes those that the wave kernel leaves.
    const uint32_t *list = nullptr, *list_count = nullptr;
    const bool few = main_tw.slots < g->num_cus &&
                     (int64_t)theta >= (g->seed_edges >= 32 ? 16 : 32) * (int64_t)main_tw.slots;
    if (!tree || few || many_small(g, theta, main_tw.slots, false)) {
        imin::SmallArgs s;
        std::memset(&s, 0, sizeof(s));
        s.inst = g->d_inst;
        s.ninst = 1;
        s.total = theta;
        s.round = 0;
        small_shape(s, g->small_launch);
        s.lt = g->model == IMIN_LT ? 1 : 0;
        s.next = g->d_sctrl + 0;
        s.spill_j = sj;
        s.spill_count = g->d_sctrl + 1;
        s.error = g->d_ctrl + 3;
        s.give_up = tree ? 1 : 0;
        if (!ok(imin::launch_decrease_small(s, small_grid(g->num_cus, g->small_launch), st)))
            return IMIN_EDEVICE;
        list = sj;
        list_count = g->d_sctrl + 1;
    }
    LargeTarget t{g->d_thr4, s_set, (int32_t)nseeds, reinterpret_cast<unsigned long long *>(d_counts),
                  g->d_stats, g->d_ctrl, ovf, &main_ws, &big_ws, &main_tw, &big_tw, g->d_D + n};
    rc = launch_large_on(g, t, theta, seed, list, list_count, false);
    if (rc) return rc;

    // Leave the graph's thresholds as created.
    if (!ok(imin::launch_mask_list(thr, g->mask_rec(), orig, g->d_in_ptr, g->d_in_edge, s_set, (int32_t)nseeds,
                                   1, st)))
        return IMIN_EDEVICE;
    if (blocked) {
        hipLaunchKernelGGL(mask_marked_kernel, dim3(grid_of(n)), dim3(kBlock), 0, st, thr, g->mask_rec(), orig,
                           g->d_in_ptr, g->d_in_edge, marks, (int32_t)n, 1);
        if (!ok(hipGetLastError())) return IMIN_EDEVICE;
    }
    unsigned long long sts[kStats];
    uint32_t ctrl[4];
    if (!ok(hipMemcpyAsync(sts, g->d_stats, sizeof(sts), hipMemcpyDeviceToHost, st)) ||
        !ok(hipMemcpyAsync(ctrl, g->d_ctrl, sizeof(ctrl), hipMemcpyDeviceToHost, st)) ||
        !ok(hipEventRecord(g->ev1, st)) || !ok(hipEventSynchronize(g->ev1)))
        return IMIN_EDEVICE;
    g->mask_known = true;
    if (ctrl[3] != 0) return IMIN_EDEVICE;
    if (stats) {
        float ms = 0.0f;
        if (!ok(hipEventElapsedTime(&ms, g->ev0, g->ev1))) return IMIN_EDEVICE;
        stats->samples = sts[0];
        stats->reached = sts[1];
        stats->edges_scanned = sts[2];
        stats->live_edges = sts[3];
        stats->spilled = sts[4];
        stats->wave_samples = sts[5];
        stats->pack_samples = sts[6];
        stats->device_ms = ms;
        stats->kernel_ms = ms;
    }
    return IMIN_OK;
}

}  // extern "C"
