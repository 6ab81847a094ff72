// api.cpp -- host side of libimin: validation, device residency of the graph, scratch
// sizing, and the greedy drivers (Algorithms 3 and 4 of arXiv 2302.13529) as device-side
// round loops. Every step of the estimate runs in the kernels of decrease.hip/select.hip.
#include "graph.h"

#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

using imin::DecreaseArgs;
using imin::Workspace;



namespace imin {
namespace host {

constexpr uint32_t kSpillSlots = 2;
constexpr int32_t kDefaultSmallWavesPerCu = 20;
constexpr int32_t kDefaultQuadLimit = 2048;
constexpr int32_t kDefaultPickDiv = 4;
// Packed kernel: a frontier vertex with more edge quads than this hands its sample over.
constexpr int32_t kDefaultPackQuadLimit = 256;
// Packed kernel workgroups per compute unit (kPackWaves waves of kPackG samples each): its
// registers allow 4 waves per SIMD, that is 4 workgroups.
constexpr int kPackGroupsPerCu = 4;

int pack_grid(int num_cus, const imin_launch &l)
{
    return std::max(1, num_cus) * (l.pack_per_cu > 0 ? l.pack_per_cu : kPackGroupsPerCu);
}
// In automatic mode the wave kernel is dropped for a graph once fewer than this share of
// a round's samples finished in it.
constexpr double kSmallKeepShare = 0.5;
// Workgroup-kernel slots while the wave kernel takes the samples first (it leaves few); a
// call whose first round leaves more than that grows them to the full count for the graph.
constexpr int32_t kSmallModeSlots = 64;


// ceil(p * 2^24) for p in [0, 1]; the product by a power of two is exact in fp32.
uint32_t live_threshold(float p)
{
    if (p <= 0.0f) return 0u;
    if (p >= 1.0f) return 1u << 24;
    return (uint32_t)std::ceil(p * 16777216.0f);
}


void free_ws(Workspace &ws)
{
    dfree(ws.map);
    dfree(ws.loc);
    dfree(ws.lvl);
    dfree(ws.extra);
    dfree(ws.rng);
    dfree(ws.epoch);
    dfree(ws.dirty);
    ws = Workspace();
}

size_t slot_bytes(int64_t n, int64_t lcap, int64_t xcap)
{
    return (size_t)n * sizeof(unsigned long long) + (size_t)lcap * sizeof(imin::LocalVtx) +
           (size_t)(lcap + 1) * sizeof(int32_t) + (size_t)xcap * sizeof(int2) + 2 * sizeof(uint32_t) +
           (size_t)lcap * sizeof(int2);
}

int alloc_ws(Workspace &ws, int64_t n, int32_t slots, int64_t lcap, int64_t xcap,
             hipStream_t stream)
{
    if (ws.slots == slots && ws.n == n && ws.lcap == lcap && ws.xcap == xcap) return IMIN_OK;
    free_ws(ws);
    // the map's local-id field holds lid + 1 <= lcap, and leaves at least one epoch bit
    int32_t lbits = 1;
    while (lbits < 32 && (int64_t(1) << lbits) <= lcap) ++lbits;
    if (lbits > 31) return IMIN_ERANGE;
    const size_t S = (size_t)slots;
    bool good = ok(hipMalloc(&ws.map, S * (size_t)n * sizeof(unsigned long long))) &&
                ok(hipMalloc(&ws.loc, S * (size_t)lcap * sizeof(imin::LocalVtx))) &&
                ok(hipMalloc(&ws.lvl, S * (size_t)(lcap + 1) * sizeof(int32_t))) &&
                ok(hipMalloc(&ws.extra, S * (size_t)std::max<int64_t>(xcap, 1) * sizeof(int2))) &&
                ok(hipMalloc(&ws.rng, S * (size_t)lcap * sizeof(int2))) &&
                ok(hipMalloc(&ws.epoch, S * sizeof(uint32_t))) &&
                ok(hipMalloc(&ws.dirty, S * sizeof(uint32_t)));
    if (!good) {
        free_ws(ws);
        (void)hipGetLastError();
        return IMIN_ENOMEM;
    }
    if (!ok(hipMemsetAsync(ws.map, 0, S * (size_t)n * sizeof(unsigned long long), stream)) ||
        !ok(hipMemsetAsync(ws.epoch, 0, S * sizeof(uint32_t), stream)) ||
        !ok(hipMemsetAsync(ws.dirty, 0, S * sizeof(uint32_t), stream))) {
        free_ws(ws);
        return IMIN_EDEVICE;
    }
    ws.slots = slots;
    ws.n = n;
    ws.lcap = lcap;
    ws.xcap = xcap;
    ws.lbits = lbits;
    ws.bytes = S * slot_bytes(n, lcap, xcap);
    return IMIN_OK;
}

void free_tree(imin::TreeWs &ws)
{
    dfree(ws.base);
    ws = imin::TreeWs();
}

size_t carve_tree(imin::TreeWs &ws, unsigned char *base, int32_t slots, int64_t lcap,
                  int64_t xcap, int64_t nclaim, int64_t words)
{
    size_t at = 0;
    auto take = [&](auto *&p, int64_t per_slot) {
        using T = typename std::remove_reference<decltype(*p)>::type;
        at = (at + 255) & ~size_t(255);
        p = base ? reinterpret_cast<T *>(base + at) : nullptr;
        at += (size_t)slots * (size_t)std::max<int64_t>(per_slot, 1) * sizeof(T);
    };
    ws.slots = slots;
    ws.lcap = lcap;
    ws.xcap = xcap;
    ws.nclaim = nclaim;
    ws.words = words;
    take(ws.planes, imin::kTreePlanes * words);
    take(ws.used, 1);
    take(ws.rng, lcap);
    take(ws.rid, lcap);
    take(ws.par, lcap);
    take(ws.acc, lcap);
    take(ws.lvl, lcap + 1);
    take(ws.extra, xcap);
    return at;
}

void free_forest(imin::ForestWs &ws)
{
    dfree(ws.base);
    ws = imin::ForestWs();
}

int alloc_forest(imin::ForestWs &ws, int32_t slots, const imin::ForestShape &shape, int64_t words,
                 hipStream_t stream)
{
    const int64_t entries = shape.entries;
    if (ws.base && ws.slots >= slots && ws.entries == entries && ws.words == words) return IMIN_OK;
    free_forest(ws);
    const size_t S = (size_t)slots, o_planes = S * (size_t)entries * 4;
    const size_t planes = S * imin::kTreePlanes * (size_t)words * 4;
    if (!ok(hipMalloc(&ws.base, o_planes + planes + S * 4))) {
        (void)hipGetLastError();
        ws.base = nullptr;
        return IMIN_ENOMEM;
    }
    ws.slots = slots;
    ws.entries = entries;
    ws.words = words;
    ws.parent = reinterpret_cast<uint32_t *>(ws.base);
    ws.planes = reinterpret_cast<uint32_t *>(ws.base + o_planes);
    ws.used = reinterpret_cast<uint32_t *>(ws.base + o_planes + planes);
    if (words > 0 && !ok(hipMemsetAsync(ws.planes, 0, planes, stream))) {
        free_forest(ws);
        return IMIN_EDEVICE;
    }
    return IMIN_OK;
}

// The wave-per-sample form's scratch.
int ensure_leaf(unsigned char *&leaf, int num_cus)
{
    if (leaf) return IMIN_OK;
    if (!ok(hipMalloc(&leaf, (size_t)imin::leaf_slots(num_cus) * imin::leaf_slot_bytes()))) {
        (void)hipGetLastError();
        leaf = nullptr;
        return IMIN_ENOMEM;
    }
    return IMIN_OK;
}

// reach_bytes: space from the row ranges on, at least.
int alloc_tree(imin::TreeWs &ws, int32_t slots, int64_t lcap, int64_t xcap, int64_t nclaim,
               int64_t words, hipStream_t stream, size_t reach_bytes = 0)
{
    if (ws.base && ws.slots == slots && ws.lcap == lcap && ws.xcap == xcap &&
        ws.nclaim == nclaim && ws.words == words && ws.reach_bytes >= reach_bytes)
        return IMIN_OK;
    reach_bytes = std::max(reach_bytes, ws.reach_bytes);
    free_tree(ws);
    imin::TreeWs w;
    size_t bytes = carve_tree(w, nullptr, slots, lcap, xcap, nclaim, words);
    unsigned char *base = nullptr;
    // the arrays ahead of the row ranges end here
    const size_t ahead = carve_tree(w, nullptr, slots, 0, 0, 0, words);
    bytes = std::max(bytes, ahead + reach_bytes);
    if (!ok(hipMalloc(&base, std::max<size_t>(bytes, 256)))) {
        (void)hipGetLastError();
        return IMIN_ENOMEM;
    }
    carve_tree(w, base, slots, lcap, xcap, nclaim, words);
    w.base = base;
    w.bytes = bytes;
    w.reach_bytes = reach_bytes;
    ws = w;
    // the planes start at zero; every launch leaves them so once they are drained
    if (slots > 0 && !ok(hipMemsetAsync(ws.planes, 0,
                                        (size_t)slots * imin::kTreePlanes * (size_t)words * 4, stream))) {
        free_tree(ws);
        return IMIN_EDEVICE;
    }
    return IMIN_OK;
}

// Per-slot scratch: every local array holds all n vertices plus the root, so only the
// extra-edge list can overflow. Its default capacity covers a quarter of the vertices; a
// graph whose m is below that can never overflow and needs no spill path.
bool small_enabled(const imin_graph *g);

// max_slots > 0 caps a new allocation (an existing one of the right shape is kept).
int size_workspaces(imin_graph *g, int32_t max_slots, uint32_t theta, bool reach_only)
{
    if (forest_on(g) && !small_enabled(g)) {
        const int32_t slots = g->force_slots > 0 ? g->force_slots : g->fshape.per_cu * g->num_cus;
        const int rc = alloc_forest(g->fws, slots, g->fshape, ((int64_t)g->nreach + 31) / 32, g->stream);
        return rc ? rc : ensure_leaf(g->leaf, g->num_cus);
    }
    if (tree_on(g)) {
        imin::tree_shape(tree_fit(g, theta, reach_only), g->shape);
        // every reachable vertex and the root fit; only the extra-edge list can overflow (its
        // capacity follows n, not the reach ids: see extra_cap)
        const int64_t lcap = (int64_t)g->nreach + 1, xmax = (int64_t)g->m + 1;
        const int64_t words = ((int64_t)g->nreach + 31) / 32;
        const bool lt = g->model == IMIN_LT;
        const int64_t nclaim = lt ? 0 : g->nclaim;
        const int64_t xcap = lt                    ? 1
                             : g->force_xcap > 0 ? std::min(g->force_xcap, xmax)
                                                 : extra_cap(g->n, g->m);
        // as many slots as can run, and no more than a call of about so many samples fills
        int64_t filled = 2 * (int64_t)g->num_cus;
        while (filled < (int64_t)theta) filled *= 2;
        const int32_t most = (int32_t)std::min<int64_t>((int64_t)g->shape.per_cu * g->num_cus, filled);
        const imin::TreeWs &have = g->main_tw;
        if (reach_only) {
            // Row ranges and level starts are all that reachability writes: a slot takes 12 bytes a
            // reach id where dominators take 25, and the many small workgroups share the space of
            // the fewer large ones of the other calls. More than two a compute unit take a
            // sixteenth of the device's memory at most. (8 bytes, with the level starts left out by
            // a test in the kernel, cost the dominators' calls 0.8 %: 22.6 ms for 22.4.)
            const size_t per = (size_t)lcap * sizeof(int2) + (size_t)(lcap + 1) * sizeof(int32_t);
            const int64_t there =
                have.base ? (int64_t)((size_t)(have.base + have.bytes -
                                               reinterpret_cast<unsigned char *>(have.rng)) / per) : 0;
            int64_t want = g->force_slots > 0 ? g->force_slots : most;
            if (there < want && g->force_slots <= 0) {
                size_t free_b = 0, total_b = 0;
                if (!ok(hipMemGetInfo(&free_b, &total_b))) return IMIN_EDEVICE;
                want = std::min<int64_t>(want, std::max<size_t>(1, ((free_b + have.bytes) / 2) / per));
                want = std::min<int64_t>(want, std::max<size_t>(2 * (size_t)g->num_cus, total_b / 16 / per));
                if (max_slots > 0) want = std::min<int64_t>(want, max_slots);
                want = std::max(want, there);
            }
            if (there < want) {
                const int rc = alloc_tree(g->main_tw, have.slots, lcap, have.slots > 0 ? have.xcap : xcap,
                                          nclaim, words, g->stream, (size_t)want * per);
                if (rc) return rc;
            }
            g->reach_tw = imin::TreeWs();
            g->reach_tw.slots = (int32_t)want;
            g->reach_tw.lcap = lcap;
            g->reach_tw.rng = g->main_tw.rng;
            g->reach_tw.lvl = reinterpret_cast<int32_t *>(g->reach_tw.rng + want * lcap);
            return IMIN_OK;
        }
        int32_t slots = g->force_slots;
        if (slots <= 0 && have.base && have.lcap == lcap && have.xcap == xcap && have.slots >= most)
            slots = have.slots;  // as many as can run: the free memory does not matter
        if (slots <= 0) {
            size_t free_b = 0, total_b = 0;
            if (!ok(hipMemGetInfo(&free_b, &total_b))) return IMIN_EDEVICE;
            free_b += g->main_tw.bytes;
            imin::TreeWs one;
            const size_t per = carve_tree(one, nullptr, 1, lcap, xcap, nclaim, words);
            const size_t by_mem = std::max<size_t>(1, (free_b / 2) / per);
            slots = (int32_t)std::min<size_t>((size_t)most, by_mem);
            if (max_slots > 0) slots = std::min(slots, max_slots);
            // an allocation that is at least as large stays
            if (g->main_tw.base && g->main_tw.lcap == lcap && g->main_tw.xcap == xcap)
                slots = std::max(slots, g->main_tw.slots);
        }
        int rc = alloc_tree(g->main_tw, slots, lcap, xcap, nclaim, words, g->stream);
        if (rc) return rc;
        if (!lt && xcap < xmax)
            return alloc_tree(g->big_tw, kSpillSlots, lcap, xmax, nclaim, 0, g->stream);
        free_tree(g->big_tw);
        return IMIN_OK;
    }
    const int64_t lcap = (int64_t)g->n + 1;
    const int64_t xmax = (int64_t)g->m + 1;
    const int64_t xcap =
        g->force_xcap > 0 ? std::min(g->force_xcap, xmax) : extra_cap(g->n, g->m);
    int32_t slots = g->force_slots;
    if (slots <= 0) {
        size_t free_b = 0, total_b = 0;
        if (!ok(hipMemGetInfo(&free_b, &total_b))) return IMIN_EDEVICE;
        free_b += g->main_ws.bytes;  // the current allocation is released before a new one
        const size_t per = slot_bytes(g->n, lcap, xcap);
        const size_t by_mem = std::max<size_t>(1, (free_b / 2) / per);
        slots = (int32_t)std::min<size_t>((size_t)imin::kSlotsPerCu * g->num_cus, by_mem);
        if (max_slots > 0) slots = std::min(slots, max_slots);
        // keep a working allocation that is at least as large, or a full-size one that the
        // free memory now sizes slightly differently
        const int32_t have = g->main_ws.slots;
        if (have > 0 && g->main_ws.lcap == lcap && g->main_ws.xcap == xcap &&
            (have >= slots || (max_slots == 0 && have > kSmallModeSlots)))
            slots = have;
    }
    int rc = alloc_ws(g->main_ws, g->n, slots, lcap, xcap, g->stream);
    if (rc) return rc;
    if (xcap < xmax) {
        rc = alloc_ws(g->big_ws, g->n, kSpillSlots, lcap, xmax, g->stream);
        if (rc) return rc;
    } else {
        free_ws(g->big_ws);
    }
    return IMIN_OK;
}

int prepare_workspaces(imin_graph *g, uint32_t theta, bool reach_only = false)
{
    const int rc = size_workspaces(g, small_enabled(g) ? kSmallModeSlots : 0, theta, reach_only);
    if (!rc && g->small_mode == -1 && tree_on(g) && !forest_on(g))
        g->wave_first = many_small(
            g, theta,
            std::min((reach_only ? g->reach_tw : g->main_tw).slots, g->shape.per_cu * g->num_cus),
            reach_only);
    return rc;
}

int ensure_ovf(imin_graph *g, uint32_t theta)
{
    if (theta <= g->ovf_cap) return IMIN_OK;
    dfree(g->d_ovf);
    if (!ok(hipMalloc(&g->d_ovf, (size_t)theta * sizeof(uint32_t)))) {
        g->ovf_cap = 0;
        return IMIN_ENOMEM;
    }
    g->ovf_cap = theta;
    return IMIN_OK;
}

int ensure_sj(imin_graph *g, uint32_t theta)
{
    if (theta <= g->sj_cap) return IMIN_OK;
    dfree(g->d_sj);
    if (!ok(hipMalloc(&g->d_sj, (size_t)theta * sizeof(uint32_t)))) {
        g->sj_cap = 0;
        return IMIN_ENOMEM;
    }
    g->sj_cap = theta;
    return IMIN_OK;
}

bool small_enabled(const imin_graph *g)
{
    if (g->small_mode == 0) return false;
    if (g->small_mode == 1) return true;
    // automatic: the LDS-claim kernel takes small samples as well as large ones, unless there are
    // very many
    return tree_on(g) ? g->wave_first : !g->small_auto_off;
}

int small_grid(int num_cus, const imin_launch &l)
{
    const int32_t wpc = l.waves_per_cu > 0 ? l.waves_per_cu : kDefaultSmallWavesPerCu;
    const int per_cu = std::max(1, (wpc + imin::kSmallWaves - 1) / imin::kSmallWaves);
    return num_cus * per_cu;
}

// The wave-kernel arguments that come from the launch shape.
void small_shape(imin::SmallArgs &s, const imin_launch &l)
{
    s.quad_limit = l.quad_limit > 0 ? l.quad_limit : kDefaultQuadLimit;
    s.pick_div = l.pick_div > 0 ? l.pick_div : kDefaultPickDiv;
}

bool launch_ok(const imin_launch *l)
{
    return !l || (l->waves_per_cu >= 0 && l->quad_limit >= 0 && l->pick_div >= 0 &&
                  (l->graph == 0 || l->graph == 1) && l->pack_per_cu >= -1);
}

int ensure_B(imin_graph *g, int32_t b)
{
    if (b <= g->B_cap) return IMIN_OK;
    dfree(g->d_B);
    if (!ok(hipMalloc(&g->d_B, (size_t)std::max(b, 1) * sizeof(int32_t)))) {
        g->B_cap = 0;
        return IMIN_ENOMEM;
    }
    g->B_cap = b;
    return IMIN_OK;
}

// Validated seed set: distinct seeds ascending, and the seed bitmap.
int seed_setup(imin_graph *g, const int32_t *S, int32_t nS, std::vector<int32_t> &seeds,
               std::vector<uint32_t> &inelig)
{
    if (!S || nS <= 0) return IMIN_EINVAL;
    inelig.assign((size_t)g->words, 0u);
    seeds.clear();
    for (int32_t i = 0; i < nS; ++i) {
        const int32_t s = S[i];
        if (s < 0 || s >= g->n) return IMIN_EINVAL;
        if (!((inelig[s >> 5] >> (s & 31)) & 1u)) {
            inelig[s >> 5] |= 1u << (s & 31);
            seeds.push_back(s);
        }
    }
    std::sort(seeds.begin(), seeds.end());
    return IMIN_OK;
}

// The graph as one instance of a wave-kernel launch (host copy in g->h_inst).
void describe(imin_graph *g, int32_t nseeds, uint64_t seed, uint32_t theta)
{
    imin::InstanceDesc &I = g->h_inst;
    I.row_ptr = g->d_row_ptr;
    I.col4 = g->d_col4;
    I.edge = g->d_edge;
    I.thr4 = g->d_thr4;
    I.lo4 = g->d_lo4;
    I.tl = g->d_tl;
    I.in_ptr = g->d_in_ptr;
    I.in_edge = g->d_in_edge;
    I.inelig = g->d_inelig;
    I.seeds = g->d_seeds;
    I.D = g->d_D;
    I.stats = g->d_stats;
    I.B = g->d_B;
    I.x = g->d_x;
    I.thr_orig = g->d_thr_orig;
    I.ctrl = g->d_ctrl;
    I.cand = g->d_cand;
    I.gr_k = -1;
    I.step = 0;
    I.nseeds = nseeds;
    I.n = g->n;
    I.nquads = (int32_t)std::max<int64_t>(((int64_t)g->m + 3) / 4, 1);
    I.nclaim = g->nclaim;
    I.nreach = g->nreach;
    I.tedge = g->d_tedge;
    I.rec = g->mask_rec();
    I.code = g->d_code;
    I.rid_vtx = g->d_rid_vtx;
    I.fnode = g->d_fnode;
    I.fin16 = g->d_fin16;
    I.fbound = g->d_fbound;
    I.fsrc = g->d_fsrc;
    I.rid_of = g->d_rid_of;
    I.nsrc = g->nsrc;
    I.seed_lo = (uint32_t)seed;
    I.seed_hi = (uint32_t)(seed >> 32);
    I.theta = theta;
    I.sample_base = 0;
}

// The vertices whose bit is set, ascending, appended to out (a word at a time).
void append_set_bits(const std::vector<uint32_t> &bits, std::vector<int32_t> &out)
{
    for (size_t w = 0; w < bits.size(); ++w) {
        uint32_t x = bits[w];
        while (x) {
            out.push_back((int32_t)(w * 32 + (size_t)__builtin_ctz(x)));
            x &= x - 1;
        }
    }
}

// The pinned block of a call that sends so much and returns nb blockers and, if counted, n counts.
int pin_call(imin_graph *g, size_t nseeds, size_t nundo, size_t nmask, int32_t nb, bool counted)
{
    if (g->in_flight) {  // a call that failed half-way: its kernels may still read the block
        if (!ok(hipStreamSynchronize(g->stream))) return IMIN_EDEVICE;
        g->in_flight = false;
    }
    auto carve = [&](unsigned char *base) {
        size_t used = 0;
        auto take = [&](size_t bytes) {
            unsigned char *p = base + used;
            used += (bytes + 255) / 256 * 256;
            return p;
        };
        imin::host::CallPin &c = g->at;
        c.inst = reinterpret_cast<imin::InstanceDesc *>(take(sizeof(imin::InstanceDesc)));
        c.stats = reinterpret_cast<unsigned long long *>(take(kCallStats * 8));
        c.ctrl = reinterpret_cast<uint32_t *>(take(16));
        c.x = reinterpret_cast<int32_t *>(take(4));
        c.seeds = reinterpret_cast<int32_t *>(take(nseeds * 4));
        c.undo = reinterpret_cast<int32_t *>(take(nundo * 4));
        c.mask = reinterpret_cast<int32_t *>(take(nmask * 4));
        c.B = reinterpret_cast<int32_t *>(take((size_t)nb * 4));
        c.inelig = reinterpret_cast<uint32_t *>(take((size_t)g->words * 4));
        c.cand = reinterpret_cast<uint32_t *>(take((size_t)g->words * 4));
        c.D = reinterpret_cast<unsigned long long *>(take(counted ? (size_t)g->n * 8 : 0));
        return used;
    };
    const size_t need = carve(nullptr);
    if (need > g->pin_cap) {
        if (g->pin) (void)hipHostFree(g->pin);
        g->pin = nullptr;
        g->pin_cap = 0;
        void *p = nullptr;
        if (!ok(hipHostMalloc(&p, need + need / 4, hipHostMallocDefault))) {
            (void)hipGetLastError();
            return IMIN_ENOMEM;
        }
        g->pin = static_cast<unsigned char *>(p);
        g->pin_cap = need + need / 4;
    }
    carve(g->pin);
    return IMIN_OK;
}

// Counts of at most so many vertices return through the pinned block (64 MiB); more are copied
// by the runtime.
constexpr int32_t kPinnedCounts = 8 << 20;

bool pinned_counts(const imin_graph *g) { return g->n <= kPinnedCounts; }

// The call's inputs to the device. cand: GreedyReplace's candidates, or null.
int upload_call_state(imin_graph *g, const std::vector<int32_t> &seeds,
                      const std::vector<uint32_t> &inelig, const std::vector<uint32_t> *cand,
                      uint64_t seed, uint32_t theta, int32_t nb, bool counted)
{
    // Working thresholds: restore the in-edges the previous call masked (all of them when
    // that call stopped half-way), then mask the in-edges of this call's seeds and blocked
    // vertices.
    uint32_t *thr = reinterpret_cast<uint32_t *>(g->d_thr4);
    const uint32_t *orig = reinterpret_cast<const uint32_t *>(g->d_thr_orig);
    g->mask_prev.swap(g->masked);
    const bool known = g->mask_known;
    g->mask_known = false;
    g->masked.clear();
    append_set_bits(inelig, g->masked);
    if (!known) {
        const int64_t quads = std::max<int64_t>(((int64_t)g->m + 3) / 4, 1);
        if (!ok(hipMemcpyAsync(g->d_thr4, g->d_thr_orig, (size_t)quads * sizeof(uint4),
                               hipMemcpyDeviceToDevice, g->stream)) ||
            (g->mask_rec() && !ok(imin::launch_edge_restore(orig, g->m, g->mask_rec(), g->stream))))
            return IMIN_EDEVICE;
        g->mask_prev.clear();
    }
    const int rc = pin_call(g, seeds.size(), g->mask_prev.size(), g->masked.size(), nb,
                            counted && pinned_counts(g));
    if (rc) return rc;
    describe(g, (int32_t)seeds.size(), seed, theta);
    const imin::host::CallPin &c = g->at;
    *c.inst = g->h_inst;
    std::copy(seeds.begin(), seeds.end(), c.seeds);
    std::copy(inelig.begin(), inelig.end(), c.inelig);
    if (cand) std::copy(cand->begin(), cand->end(), c.cand);
    std::fill(c.B, c.B + nb, -1);
    std::copy(g->masked.begin(), g->masked.end(), c.mask);
    // a vertex masked in both calls stays masked: the kernel's lists have no order
    int32_t nundo = 0;
    for (int32_t v : g->mask_prev)
        if (!((inelig[v >> 5] >> (v & 31)) & 1u)) c.undo[nundo++] = v;
    imin::CallSetup s{};
    s.inst = c.inst;
    s.seeds = c.seeds;
    s.undo = c.undo;
    s.mask = c.mask;
    s.inelig = c.inelig;
    s.cand = cand ? c.cand : nullptr;
    s.nseeds = (int32_t)seeds.size();
    s.nundo = nundo;
    s.nmask = (int32_t)g->masked.size();
    s.words = (int32_t)inelig.size();
    s.nstats = kCallStats;
    s.nctrl = 4;
    s.d_inst = g->d_inst;
    s.d_seeds = g->d_seeds;
    s.d_inelig = g->d_inelig;
    s.d_cand = g->d_cand;
    s.d_stats = g->d_stats;
    s.d_ctrl = g->d_ctrl;
    s.thr = thr;
    s.rec = g->mask_rec();
    s.thr_orig = orig;
    s.in_ptr = g->d_in_ptr;
    s.in_edge = g->d_in_edge;
    g->in_flight = true;
    return ok(imin::launch_call_setup(s, g->stream)) ? IMIN_OK : IMIN_EDEVICE;
}

// The call ended with the seeds and `blockers` masked.
void end_masks(imin_graph *g, const std::vector<int32_t> &blockers)
{
    for (int32_t v : blockers) g->masked.push_back(v);
    g->mask_known = true;
}

uint32_t *thr_w(imin_graph *g) { return reinterpret_cast<uint32_t *>(g->d_thr4); }

// Rounds are timed on the device's clock, not by events.
bool round_clock(const imin_graph *g) { return tree_on(g); }

unsigned long long *clock_of(imin_graph *g) { return round_clock(g) ? g->d_stats + kClock : nullptr; }

// A fresh pair of timing events for one round's decrease launches.
int kernel_events(imin_graph *g, hipEvent_t *a, hipEvent_t *b)
{
    while (g->kev.size() < g->kev_used + 2) {
        hipEvent_t e;
        if (!ok(hipEventCreate(&e))) return IMIN_EDEVICE;
        g->kev.push_back(e);
    }
    *a = g->kev[g->kev_used];
    *b = g->kev[g->kev_used + 1];
    g->kev_used += 2;
    return IMIN_OK;
}

// The workgroup-per-sample kernel with Philox key `key` over samples 0..theta-1, or over
// the device list `list` of *count samples (at most theta), then the large-scratch launch
// for the samples that overflowed it. D and the stats accumulate: the main launch's slots
// decide one by one whether to keep reach counts in their maps (count_reach allows it),
// and the flush after the launches adds what they kept into D.
int launch_large_on(imin_graph *g, const LargeTarget &t, uint32_t theta, uint64_t key,
                    const uint32_t *list, const uint32_t *count, bool reach_only)
{
    if (tree_on(g)) {
        const bool lt = g->model == IMIN_LT;
        const bool spill = t.big_tw->slots > 0;
        imin::TreeArgs a{};
        a.row_ptr = g->d_row_ptr;
        a.edge = g->d_tedge;
        a.code = g->d_code;
        a.thr4 = t.thr4;
        a.tl = g->d_tl;
        a.seeds = t.seeds;
        a.nseeds = t.nseeds;
        a.nclaim = g->nclaim;
        a.nreach = g->nreach;
        a.rid_vtx = g->d_rid_vtx;
        a.key_lo = (uint32_t)key;
        a.key_hi = (uint32_t)(key >> 32);
        a.theta = theta;
        a.sample_list = list;
        a.sample_count = count;
        a.next = t.ctrl + 0;
        a.D = t.Dr;
        a.stats = t.stats;
        a.ovf_list = t.ovf;
        a.ovf_count = t.ctrl + 2;
        a.error = t.ctrl + 3;
        a.spill_ok = spill ? 1 : 0;
        a.reach_only = reach_only ? 1 : 0;
        a.count_reach = reach_only ? 0 : 1;
        a.ws = *t.main_tw;
        a.ws.slots = (int32_t)std::min<uint32_t>((uint32_t)t.main_tw->slots, theta);
        if (g->force_slots <= 0)
            a.ws.slots = std::min(a.ws.slots, g->shape.per_cu * g->num_cus);
        const int32_t used = a.ws.slots;
        if (!ok(imin::launch_tree(a, g->shape, lt, g->stream))) return IMIN_EDEVICE;
        if (spill && !reach_only) {
            a.sample_list = t.ovf;
            a.sample_count = t.ctrl + 2;
            a.next = t.ctrl + 1;
            a.spill_ok = 0;
            a.count_reach = 0;
            a.ws = *t.big_tw;
            if (!ok(imin::launch_tree(a, g->shape, lt, g->stream))) return IMIN_EDEVICE;
        }
        if (!reach_only && !ok(imin::launch_drain_planes(*t.main_tw, used, g->d_rid_vtx,
                                                         g->nreach, t.Dr, t.D, g->stream)))
            return IMIN_EDEVICE;
        return IMIN_OK;
    }
    const bool spill = t.big_ws->slots > 0;
    DecreaseArgs a;
    std::memset(&a, 0, sizeof(a));
    a.row_ptr = g->d_row_ptr;
    a.col4 = g->d_col4;
    a.edge = g->d_edge;
    a.thr4 = t.thr4;
    a.lo4 = g->d_lo4;
    a.tl = g->d_tl;
    a.seeds = t.seeds;
    a.nseeds = t.nseeds;
    a.n = g->n;
    a.key_lo = (uint32_t)key;
    a.key_hi = (uint32_t)(key >> 32);
    a.theta = theta;
    a.sample_list = list;
    a.sample_count = count;
    a.next = t.ctrl + 0;
    a.D = t.D;
    a.stats = t.stats;
    a.ovf_list = t.ovf;
    a.ovf_count = t.ctrl + 2;
    a.error = t.ctrl + 3;
    a.spill_ok = spill ? 1 : 0;
    a.reach_only = reach_only ? 1 : 0;
    a.count_reach = reach_only ? 0 : 1;
    a.ws = *t.main_ws;
    a.ws.slots = (int32_t)std::min<uint32_t>((uint32_t)t.main_ws->slots, theta);
    const int32_t used = a.ws.slots;
    if (!ok(imin::launch_decrease(a, g->stream))) return IMIN_EDEVICE;
    if (spill) {
        a.sample_list = t.ovf;
        a.sample_count = t.ctrl + 2;
        a.next = t.ctrl + 1;
        a.spill_ok = 0;
        a.count_reach = 0;
        a.ws = *t.big_ws;
        if (!ok(imin::launch_decrease(a, g->stream))) return IMIN_EDEVICE;
    }
    if (!reach_only && !ok(imin::launch_flush_counts(*t.main_ws, used, t.D, g->stream)))
        return IMIN_EDEVICE;
    return IMIN_OK;
}

void multi_free(MultiScratch &ms)
{
    if (ms.exec) (void)hipGraphExecDestroy(ms.exec);
    ms.exec = nullptr;
    ms.exec_key.clear();
    dfree(ms.table);
    dfree(ms.stages);
    dfree(ms.stage);
    dfree(ms.rounds);
    dfree(ms.out);
    ms.table_cap = ms.stages_cap = ms.stage_cap = ms.rounds_cap = ms.out_cap = 0;
    free_ws(ms.main_ws);
    free_ws(ms.big_ws);
    free_tree(ms.main_tw);
    free_tree(ms.big_tw);
    free_forest(ms.fws);
    free_forest(ms.low_ws);
    dfree(ms.leaf);
    dfree(ms.ctrl);
    dfree(ms.pi);
    dfree(ms.pj);
    dfree(ms.si);
    dfree(ms.sj);
    dfree(ms.oi);
    dfree(ms.oj);
    dfree(ms.part_d);
    dfree(ms.part_i);
    ms.n = ms.m = 0;
    ms.cap = 0;
    ms.inst_cap = 0;
}

void MultiSize::add(const imin_graph *g)
{
    n = std::max<int64_t>(n, g->n);
    m = std::max<int64_t>(m, g->m);
    nclaim = std::max<int64_t>(nclaim, g->nclaim);
    nreach = std::max<int64_t>(nreach, g->nreach);
    nsrc = std::max<int64_t>(nsrc, g->nsrc);
    forest = forest && g->forest;
    lt = g->model == IMIN_LT;
}

// Many-instance rounds on graphs with more reach ids than this hand their larger samples to the
// LDS-claim kernels. What decides is the number and size of the hand-overs, for which the reach
// ids only stand in. Where samples of 10^4 vertices carry the round, a workgroup of 512 threads
// pays: 48 queries on a 1M-vertex graph 211 ms without, 153 with. Where hand-overs are few, the
// 2048 smaller slots of the other kernel keep more of them in flight: 96 trivalency graphs of at
// most 100,000 vertices 13.2 ms against 13.6, 32 queries on an 8k-vertex graph 10.8 against 12.7.
// Below the line the other kernel is also kept where it loses: 48 weighted-cascade graphs of at
// most 100,000 vertices take 54.6 ms, and would take 51.0 with 512 threads and 46.2 with 256; a
// weighted-cascade GreedyReplace batch 27.1, 22.2 and 19.5; a 131k-vertex server 21.0, 20.1, 20.4.
constexpr int64_t kMultiTreeReach = 1 << 17;

// The workgroup kernel's slots for many-instance rounds: as many as a compute unit holds,
// within a quarter of the free memory.
int multi_slots(MultiScratch &ms, int num_cus, const MultiSize &size, hipStream_t stream)
{
    const int64_t max_n = size.n, max_m = size.m;
    size_t free_b = 0, total_b = 0;
    if (!ok(hipMemGetInfo(&free_b, &total_b))) return IMIN_EDEVICE;
    ms.forest = size.lt && size.forest && imin::forest_shape(size.nreach, size.nsrc, ms.fshape);
    if (ms.forest) {
        const int cus = std::max(1, num_cus);
        int rc = ensure_leaf(ms.leaf, num_cus);
        if (!rc) rc = alloc_forest(ms.fws, ms.fshape.per_cu * cus, ms.fshape, 0, stream);
        ms.split = size.nreach > imin::kForestLow &&
                   imin::forest_shape(imin::kForestLow, size.nsrc, ms.low_shape) &&
                   ms.low_shape.block < ms.fshape.block;
        if (!rc && ms.split)
            rc = alloc_forest(ms.low_ws, ms.low_shape.per_cu * cus, ms.low_shape, 0, stream);
        return rc;
    }
    const int64_t xmax = max_m + 1;
    imin::TreeFit fit;
    fit.nclaim = size.nclaim;
    fit.nreach = size.nreach;
    fit.theta = 1 << 20;
    fit.num_cus = num_cus;
    ms.tree = !size.lt && size.nreach > kMultiTreeReach && imin::tree_shape(fit, ms.shape);
    if (ms.tree) {
        int rc = ensure_leaf(ms.leaf, num_cus);
        if (rc) return rc;
        const int64_t lcap = size.nreach + 1;
        const int64_t xcap = extra_cap(max_n, max_m);
        free_b += ms.main_tw.bytes;
        imin::TreeWs one;
        const size_t per = carve_tree(one, nullptr, 1, lcap, xcap, size.nclaim, 0);
        const int32_t slots = (int32_t)std::max<size_t>(
            1, std::min<size_t>((size_t)ms.shape.per_cu * std::max(1, num_cus), (free_b / 4) / per));
        rc = alloc_tree(ms.main_tw, slots, lcap, xcap, size.nclaim, 0, stream);
        if (rc) return rc;
        if (xcap < xmax)
            return alloc_tree(ms.big_tw, (int32_t)kSpillSlots, lcap, xmax, size.nclaim, 0, stream);
        free_tree(ms.big_tw);
        return IMIN_OK;
    }
    const int64_t lcap = max_n + 1;
    const int64_t xcap = extra_cap(max_n, max_m);
    free_b += ms.main_ws.bytes;
    const size_t per = slot_bytes(max_n, lcap, xcap);
    const int32_t slots = (int32_t)std::max<size_t>(
        1, std::min<size_t>((size_t)imin::kMultiSlotsPerCu * std::max(1, num_cus),
                            (free_b / 4) / per));
    int rc = alloc_ws(ms.main_ws, max_n, slots, lcap, xcap, stream);
    if (rc) return rc;
    if (xcap < xmax) {
        rc = alloc_ws(ms.big_ws, max_n, (int32_t)kSpillSlots, lcap, xmax, stream);
        if (rc) return rc;
    } else {
        free_ws(ms.big_ws);
    }
    return IMIN_OK;
}

int multi_alloc(MultiScratch &ms, int num_cus, const MultiSize &size, uint32_t cap,
                int32_t max_inst, hipStream_t stream)
{
    const int rc = multi_slots(ms, num_cus, size, stream);
    if (rc) return rc;
    if (cap > ms.cap) {
        dfree(ms.pi);
        dfree(ms.pj);
        dfree(ms.si);
        dfree(ms.sj);
        dfree(ms.oi);
        dfree(ms.oj);
        ms.cap = 0;
        if (!ok(hipMalloc(&ms.pi, (size_t)cap * sizeof(uint32_t))) ||
            !ok(hipMalloc(&ms.pj, (size_t)cap * sizeof(uint32_t))) ||
            !ok(hipMalloc(&ms.si, (size_t)cap * sizeof(uint32_t))) ||
            !ok(hipMalloc(&ms.sj, (size_t)cap * sizeof(uint32_t))) ||
            !ok(hipMalloc(&ms.oi, (size_t)cap * sizeof(uint32_t))) ||
            !ok(hipMalloc(&ms.oj, (size_t)cap * sizeof(uint32_t)))) {
            (void)hipGetLastError();
            return IMIN_ENOMEM;
        }
        ms.cap = cap;
    }
    if (max_inst > ms.inst_cap) {
        dfree(ms.part_d);
        dfree(ms.part_i);
        ms.inst_cap = 0;
        const size_t parts = (size_t)max_inst * imin::kArgParts;
        if (!ok(hipMalloc(&ms.part_d, parts * sizeof(unsigned long long))) ||
            !ok(hipMalloc(&ms.part_i, parts * sizeof(int32_t)))) {
            (void)hipGetLastError();
            return IMIN_ENOMEM;
        }
        ms.inst_cap = max_inst;
    }
    if (!ms.ctrl && !ok(hipMalloc(&ms.ctrl, kMultiCtrl * sizeof(uint32_t)))) {
        (void)hipGetLastError();
        return IMIN_ENOMEM;
    }
    if (!ok(imin::launch_fill_u32(ms.ctrl, kMultiCtrl, 0, stream))) return IMIN_EDEVICE;
    ms.n = size.n;
    ms.m = size.m;
    return IMIN_OK;
}

int32_t gr_candidates(const imin_graph *g, const std::vector<int32_t> &seeds,
                      const std::vector<uint32_t> &inelig, std::vector<uint32_t> &cand)
{
    cand.assign((size_t)g->words, 0u);
    int32_t ncb = 0;
    for (int32_t s : seeds) {
        for (int32_t e = g->row_ptr[s]; e < g->row_ptr[s + 1]; ++e) {
            const int32_t v = g->col[e];
            const bool is_seed = (inelig[v >> 5] >> (v & 31)) & 1u;
            if (!is_seed && !((cand[v >> 5] >> (v & 31)) & 1u)) {
                cand[v >> 5] |= 1u << (v & 31);
                ++ncb;
            }
        }
    }
    return ncb;
}

int multi_round(MultiScratch &ms, const imin::InstanceDesc *inst, int32_t ninst, uint32_t total,
                uint32_t round, const imin_launch &shape, int num_cus, bool select, bool gr,
                bool lt, hipStream_t stream)
{
    if (total > ms.cap) return IMIN_ERANGE;
    // words 0-5, 7 and 8 restart every round; the error words 2 and 6 accumulate, and word 9
    // (instances done) over the call
    if (!ok(imin::launch_batch_zero(inst, ninst, stream)) ||
        !ok(imin::launch_fill_u32(ms.ctrl, 2, 0, stream)) ||
        !ok(imin::launch_fill_u32(ms.ctrl + 3, 3, 0, stream)) ||
        !ok(imin::launch_fill_u32(ms.ctrl + 7, 2, 0, stream)))
        return IMIN_EDEVICE;
    if (gr && !ok(imin::launch_batch_gr_prepare(inst, ninst, (int32_t)round, stream)))
        return IMIN_EDEVICE;
    // The smallest samples first, several to a wavefront (independent cascade only: the
    // packed kernel keeps the seed level's edge coins in registers); what outgrows it goes
    // straight to the workgroup kernel through a device-side list. The hand-overs are the
    // few larger samples (over 63 vertices or 64 extra edges), which the workgroup kernel's
    // 2048 slots finish sooner than one wavefront each would. Without the packed kernel
    // (linear threshold, or switched off) the one-sample-per-wave kernel takes every sample
    // first and hands its overflow on.
    const bool pack = !lt && shape.pack_per_cu >= 0;
    if (pack) {
        imin::PackArgs p;
        std::memset(&p, 0, sizeof(p));
        p.inst = inst;
        p.ninst = ninst;
        p.total = total;
        p.round = round;
        p.quad_limit = kDefaultPackQuadLimit;
        p.pick_div = shape.pick_div > 0 ? shape.pick_div : kDefaultPickDiv;
        p.next = ms.ctrl + 8;
        p.out_inst = ms.pi;
        p.out_j = ms.pj;
        p.out_count = ms.ctrl + 7;
        p.error = ms.ctrl + 2;
        if (!ok(imin::launch_decrease_pack(p, pack_grid(num_cus, shape), stream))) return IMIN_EDEVICE;
    }
    imin::SmallArgs s;
    std::memset(&s, 0, sizeof(s));
    s.inst = inst;
    s.ninst = ninst;
    s.total = total;
    s.round = round;
    small_shape(s, shape);
    s.lt = lt ? 1 : 0;
    s.next = ms.ctrl + 0;
    s.spill_inst = ms.si;
    s.spill_j = ms.sj;
    s.spill_count = ms.ctrl + 1;
    s.error = ms.ctrl + 2;
    // Samples that stay small go to the wave-per-sample kernel, one per wavefront: what the
    // packed kernel hands over, and under linear threshold every sample. Then the kernel for the
    // large ones; under linear threshold the smaller graphs' in workgroups sized for those.
    // Hand-overs of the packed kernel that do not give each of its wavefronts one are better off
    // in whole workgroups: with 750 a round (96 graphs, 2,000 samples each) the wave-per-sample
    // kernel takes 130 us and saves 40 behind it. With 43,000 a round (48 queries on a 1M-vertex
    // graph) it takes 0.98 ms and saves 1.68.
    const bool leaf = (ms.forest || ms.tree) && shape.pack_per_cu >= 0;
    const bool split = leaf && ms.forest && ms.split;
    const uint32_t leave = pack ? (uint32_t)imin::leaf_slots(num_cus) : 0;
    if (leaf) {
        imin::LeafArgs f{};
        f.inst = inst;
        f.ninst = ninst;
        f.total = total;
        f.round = round;
        if (pack) {
            f.sample_list = ms.pj;
            f.sample_inst = ms.pi;
            f.sample_count = ms.ctrl + 7;
            f.leave = leave;
        }
        f.next = ms.ctrl + 0;
        f.out_inst = ms.si;
        f.out_j = ms.sj;
        f.out_count = ms.ctrl + 1;
        if (split) {
            f.low_reach = imin::kForestLow;
            f.low_inst = ms.pi;
            f.low_j = ms.pj;
            f.low_count = ms.ctrl + 7;
        }
        if (!ok(imin::launch_leaf(f, ms.leaf, imin::leaf_slots(num_cus), true, lt, stream)))
            return IMIN_EDEVICE;
    } else if (!pack && !ok(imin::launch_decrease_small(s, small_grid(num_cus, shape), stream))) {
        return IMIN_EDEVICE;
    }
    if (ms.forest) {
        imin::ForestArgs f{};
        f.inst = inst;
        f.theta = total;
        f.round = round;
        if (split) {
            f.sample_list = ms.pj;
            f.sample_inst = ms.pi;
            f.sample_count = ms.ctrl + 7;
            f.next = ms.ctrl + 4;
            f.ws = ms.low_ws;
            if (!ok(imin::launch_forest(f, ms.low_shape, ms.low_ws.slots, true, stream)))
                return IMIN_EDEVICE;
        }
        f.sample_list = ms.sj;
        f.sample_inst = ms.si;
        f.sample_count = ms.ctrl + 1;
        f.next = ms.ctrl + 3;
        f.ws = ms.fws;
        if (!ok(imin::launch_forest(f, ms.fshape, ms.fws.slots, true, stream))) return IMIN_EDEVICE;
    } else if (ms.tree) {
        const bool spill = ms.big_tw.slots > 0;
        imin::TreeArgs a{};
        a.theta = total;
        a.sample_list = ms.sj;
        a.sample_inst = ms.si;
        a.sample_count = ms.ctrl + 1;
        if (leaf) {
            a.alt_list = ms.pj;
            a.alt_inst = ms.pi;
            a.alt_count = ms.ctrl + 7;
            a.alt_most = leave;
        }
        a.next = ms.ctrl + 3;
        a.ovf_list = ms.oj;
        a.ovf_count = ms.ctrl + 5;
        a.error = ms.ctrl + 6;
        a.spill_ok = spill ? 1 : 0;
        a.ws = ms.main_tw;
        a.inst = inst;
        a.ovf_inst = ms.oi;
        a.round = round;
        if (!ok(imin::launch_tree(a, ms.shape, false, stream))) return IMIN_EDEVICE;
        if (spill) {
            a.alt_count = nullptr;
            a.sample_list = ms.oj;
            a.sample_inst = ms.oi;
            a.sample_count = ms.ctrl + 5;
            a.next = ms.ctrl + 4;
            a.spill_ok = 0;
            a.ws = ms.big_tw;
            if (!ok(imin::launch_tree(a, ms.shape, false, stream))) return IMIN_EDEVICE;
        }
    } else {
        const bool spill = ms.big_ws.slots > 0;
        DecreaseArgs a;
        std::memset(&a, 0, sizeof(a));
        a.n = (int32_t)ms.n;
        a.theta = total;
        a.sample_list = pack ? ms.pj : ms.sj;
        a.sample_count = pack ? ms.ctrl + 7 : ms.ctrl + 1;
        a.next = ms.ctrl + 3;
        a.ovf_list = ms.oj;
        a.ovf_count = ms.ctrl + 5;
        a.error = ms.ctrl + 6;
        a.spill_ok = spill ? 1 : 0;
        a.ws = ms.main_ws;
        a.inst = inst;
        a.sample_inst = pack ? ms.pi : ms.si;
        a.ovf_inst = ms.oi;
        a.round = round;
        a.lt = lt ? 1 : 0;
        if (!ok(imin::launch_decrease(a, stream))) return IMIN_EDEVICE;
        if (spill) {
            a.sample_list = ms.oj;
            a.sample_inst = ms.oi;
            a.sample_count = ms.ctrl + 5;
            a.next = ms.ctrl + 4;
            a.spill_ok = 0;
            a.ws = ms.big_ws;
            if (!ok(imin::launch_decrease(a, stream))) return IMIN_EDEVICE;
        }
    }
    if (select) {
        if (ninst > ms.inst_cap) return IMIN_ERANGE;
        if (!ok(imin::launch_batch_argmax(inst, ninst, (int32_t)round, ms.part_d, ms.part_i,
                                          ms.ctrl + 9, stream)))
            return IMIN_EDEVICE;
    }
    return IMIN_OK;
}

int multi_errors(MultiScratch &ms, uint32_t *wave_err, uint32_t *wg_err, hipStream_t stream)
{
    uint32_t w[7];
    if (!ok(hipMemcpyAsync(w, ms.ctrl, sizeof(w), hipMemcpyDeviceToHost, stream)) ||
        !ok(hipStreamSynchronize(stream)))
        return IMIN_EDEVICE;
    *wave_err = w[2];
    *wg_err = w[6];
    return IMIN_OK;
}

// The graph's own call state as the target of the workgroup kernel.
int launch_large(imin_graph *g, int32_t nseeds, uint32_t theta, uint64_t key,
                 const uint32_t *list, const uint32_t *count, bool reach_only = false)
{
    LargeTarget t{g->d_thr4, g->d_seeds, nseeds, g->d_D, g->d_stats, g->d_ctrl, g->d_ovf,
                  &g->main_ws, &g->big_ws, reach_only ? &g->reach_tw : &g->main_tw, &g->big_tw,
                  g->d_D + g->n};
    return launch_large_on(g, t, theta, key, list, count, reach_only);
}

// One call of Algorithm 2 with Philox key seed + call, leaving D on the device. With the
// wave kernel on, it runs every sample first and leaves the ones that outgrow it to the
// workgroup kernel, through a device-side list (no host round trip).
// `restore`: a vertex whose in-edges are unmasked first, or -1.
int decrease_round(imin_graph *g, int32_t nseeds, uint32_t theta, uint64_t seed, uint32_t call,
                   bool reach_only = false, int32_t restore = -1)
{
    int rc = IMIN_OK;
    if (g->probe == 2) {
        // Automatic mode, a call that kept the wave kernel: after a timed round with it, a
        // timed trial round of the workgroup kernel alone, at its full slot count.
        g->small_auto_off = true;
        rc = size_workspaces(g, 0, theta, reach_only);
        if (rc) return rc;
    } else if (g->probe == 3) {
        // The call keeps whichever form ran its round faster (results are the same).
        g->probe = 0;
        const size_t a = g->probe_kev[0], b = g->probe_kev[1];
        float with = 0.0f, without = 0.0f;
        if (!ok(hipEventSynchronize(g->kev[b + 1])) ||
            !ok(hipEventElapsedTime(&with, g->kev[a], g->kev[a + 1])) ||
            !ok(hipEventElapsedTime(&without, g->kev[b], g->kev[b + 1])))
            return IMIN_EDEVICE;
        g->small_auto_off = without < with;
    }
    const bool small = small_enabled(g);
    imin::RoundSetup rs{};
    rs.D = reach_only ? nullptr : g->d_D;
    rs.count = (int64_t)g->n + g->nreach;
    rs.ctrl = g->d_ctrl;
    rs.sctrl = g->d_sctrl;
    rs.clock = g->d_stats + kClock;
    rs.restore = restore;
    rs.inelig = g->d_inelig;
    rs.thr = thr_w(g);
    rs.rec = g->mask_rec();
    rs.thr_orig = reinterpret_cast<const uint32_t *>(g->d_thr_orig);
    rs.in_ptr = g->d_in_ptr;
    rs.in_edge = g->d_in_edge;
    if (!ok(imin::launch_round_setup(rs, g->stream))) return IMIN_EDEVICE;
    // The round's time: from here to the next kernel behind the round, on the device's clock. A
    // pair of events costs a round 15 us; only the choice between the forms needs them.
    hipEvent_t k0 = nullptr, k1 = nullptr;
    if (!round_clock(g)) {
        rc = kernel_events(g, &k0, &k1);
        if (rc) return rc;
        if (g->probe == 1 || g->probe == 2) {
            g->probe_kev[g->probe - 1] = g->kev_used - 2;
            ++g->probe;
        }
        if (!ok(hipEventRecord(k0, g->stream))) return IMIN_EDEVICE;
    }
    if (forest_on(g) && !small) {
        // Linear threshold on a graph that fits the forest kernel: samples that stay small
        // first (automatic mode), then it.
        const bool leaf = g->small_mode == -1;
        if (leaf) {
            imin::LeafArgs f{};
            f.inst = g->d_inst;
            f.ninst = 1;
            f.total = theta;
            f.round = call;
            f.reach_only = reach_only ? 1 : 0;
            f.next = g->d_sctrl + 0;
            f.out_j = g->d_sj;
            f.out_count = g->d_sctrl + 1;
            if (!ok(imin::launch_leaf(f, g->leaf,
                                      (int)std::min<uint32_t>(theta, (uint32_t)imin::leaf_slots(g->num_cus)),
                                      false, true, g->stream)))
                return IMIN_EDEVICE;
        }
        imin::ForestArgs f{};
        f.inst = g->d_inst;
        f.theta = theta;
        f.round = call;
        f.sample_list = leaf ? g->d_sj : nullptr;
        f.sample_count = g->d_sctrl + 1;
        f.next = g->d_sctrl + 2;
        f.reach_only = reach_only ? 1 : 0;
        f.Dr = g->d_D + g->n;
        f.ws = g->fws;
        int32_t slots = g->force_slots > 0 ? g->force_slots : g->fshape.per_cu * g->num_cus;
        slots = (int32_t)std::min<uint32_t>(theta, (uint32_t)slots);
        if (!ok(imin::launch_forest(f, g->fshape, slots, false, g->stream))) return IMIN_EDEVICE;
        if (!reach_only) {
            imin::TreeWs counted;
            counted.planes = g->fws.planes;
            counted.used = g->fws.used;
            counted.words = g->fws.words;
            if (!ok(imin::launch_drain_planes(counted, slots, g->d_rid_vtx, g->nreach, g->d_D + g->n,
                                              g->d_D, g->stream)))
                return IMIN_EDEVICE;
        }
        return IMIN_OK;
    }
    if (small) {
        imin::SmallArgs s;
        std::memset(&s, 0, sizeof(s));
        s.inst = g->d_inst;
        s.ninst = 1;
        s.total = theta;
        s.round = call;
        small_shape(s, g->small_launch);
        s.reach_only = reach_only ? 1 : 0;
        s.lt = g->model == IMIN_LT ? 1 : 0;
        s.next = g->d_sctrl + 0;
        s.spill_inst = nullptr;
        s.spill_j = g->d_sj;
        s.spill_count = g->d_sctrl + 1;
        s.error = g->d_ctrl + 3;
        s.give_up = g->wave_first ? 1 : 0;
        if (!ok(imin::launch_decrease_small(s, small_grid(g->num_cus, g->small_launch),
                                            g->stream)))
            return IMIN_EDEVICE;
        if (g->auto_pending) {
            // First round of the call. When the wave kernel handed over more samples than
            // the workgroup kernel has slots, that kernel gets its full slot count now (the
            // samples it receives are the large ones). In automatic mode, when it handed
            // over most samples, the wave kernel also sits out the call's later rounds.
            // Results are the same either way.
            g->auto_pending = false;
            uint32_t handed = 0;
            if (!ok(hipMemcpyAsync(&handed, g->d_sctrl + 1, sizeof(handed),
                                   hipMemcpyDeviceToHost, g->stream)) ||
                !ok(hipStreamSynchronize(g->stream)))
                return IMIN_EDEVICE;
            const bool drop = g->small_mode == -1 &&
                              (double)handed > (1.0 - kSmallKeepShare) * (double)theta;
            if (drop) g->small_auto_off = true;
            if (drop) g->wave_first = false;
            if (g->small_mode == -1 && !drop && !reach_only && !tree_on(g)) {
                // kept: the next round is timed with the wave kernel (this one waited for
                // the host), the one after it without
                g->probe = 1;
            }
            const int32_t slots = !tree_on(g)  ? g->main_ws.slots
                                  : reach_only ? g->reach_tw.slots
                                               : g->main_tw.slots;
            if (drop || handed > (uint32_t)slots) {
                rc = size_workspaces(g, 0, theta, reach_only);
                if (rc) return rc;
            }
        }
        rc = launch_large(g, nseeds, theta, seed + call, g->d_sj, g->d_sctrl + 1, reach_only);
    } else {
        rc = launch_large(g, nseeds, theta, seed + call, nullptr, nullptr, reach_only);
    }
    if (rc) return rc;
    if (k1 && !ok(hipEventRecord(k1, g->stream))) return IMIN_EDEVICE;
    return IMIN_OK;
}

// Returns the stats, the error flag and the counts (D: null, or the device's, which go to the
// pinned block) and waits; IMIN_EDEVICE if a sample was lost. last_round: the call's last round
// is still to be timed.
int finish_call(imin_graph *g, imin_stats *stats, const unsigned long long *D, bool last_round)
{
    const unsigned long long *st = g->at.stats;
    if (!ok(imin::launch_call_result(D, g->n, g->at.D, g->d_stats, kCallStats, g->at.stats, g->d_ctrl,
                                     4, g->at.ctrl, last_round ? clock_of(g) : nullptr, g->stream)) ||
        !ok(hipEventRecord(g->ev1, g->stream)) || !ok(hipEventSynchronize(g->ev1)))
        return IMIN_EDEVICE;
    g->in_flight = false;
    if (g->at.ctrl[3] != 0) return IMIN_EDEVICE;
    if (stats) {
        float ms = 0.0f;
        if (!ok(hipEventElapsedTime(&ms, g->ev0, g->ev1))) return IMIN_EDEVICE;
        stats->samples = st[0];
        stats->reached = st[1];
        stats->edges_scanned = st[2];
        stats->live_edges = st[3];
        stats->spilled = st[4];
        stats->wave_samples = st[5];
        stats->pack_samples = st[6];
        stats->device_ms = ms;
        double kms = (double)st[kClock + 1] / (double)g->clock_khz;
        for (size_t i = 0; i + 1 < g->kev_used; i += 2) {
            float x = 0.0f;
            if (!ok(hipEventElapsedTime(&x, g->kev[i], g->kev[i + 1]))) return IMIN_EDEVICE;
            kms += x;
        }
        stats->kernel_ms = kms;
    }
    return IMIN_OK;
}

int begin_call(imin_graph *g, const std::vector<int32_t> &seeds)
{
    if (!ok(hipSetDevice(g->device))) return IMIN_EDEVICE;
    g->kev_used = 0;
    g->small_auto_off = false;  // every call tries the wave kernel in its first round
    g->auto_pending = true;
    g->probe = 0;
    g->wave_first = false;
    g->prefer = 0;
    g->seed_edges = out_edges(g, seeds.data(), seeds.size());
    if (!ok(hipEventRecord(g->ev0, g->stream))) return IMIN_EDEVICE;
    return IMIN_OK;
}

// A greedy call's first two rounds are on their way: the later ones' workgroup size by the first
// one's samples, whose counters come back while the second runs.
int fit_rounds(imin_graph *g, int32_t round, uint32_t theta)
{
    if (round > 1 || !tree_on(g) || g->model == IMIN_LT || g->force_block || small_enabled(g))
        return IMIN_OK;
    if (round == 0)
        return ok(imin::launch_call_result(nullptr, 0, nullptr, g->d_stats, kCallStats, g->at.stats,
                                           g->d_ctrl, 4, g->at.ctrl, nullptr, g->stream)) &&
                       ok(hipEventRecord(g->ev1, g->stream))
                   ? IMIN_OK
                   : IMIN_EDEVICE;
    if (!ok(hipEventSynchronize(g->ev1))) return IMIN_EDEVICE;
    g->prefer = imin::block_after(tree_fit(g, theta, false), (double)g->at.stats[1] / (double)theta,
                                  g->at.stats[imin::kStatLargest]);
    if (!g->prefer) return IMIN_OK;
    // the second round still runs in the scratch that this may replace
    if (!ok(hipStreamSynchronize(g->stream))) return IMIN_EDEVICE;
    return size_workspaces(g, 0, theta, false);
}

void destroy(imin_graph *g)
{
    if (!g) return;
    (void)hipSetDevice(g->device);
    if (g->stream) (void)hipStreamSynchronize(g->stream);
    if (g->batch_ms) {
        multi_free(*g->batch_ms);
        delete g->batch_ms;
        g->batch_ms = nullptr;
    }
    free_ws(g->main_ws);
    free_ws(g->big_ws);
    free_tree(g->main_tw);
    free_tree(g->big_tw);
    free_forest(g->fws);
    dfree(g->leaf);
    dfree(g->block);
    dfree(g->d_sj);
    dfree(g->d_ovf);
    dfree(g->d_B);
    if (g->pin) (void)hipHostFree(g->pin);
    for (hipEvent_t e : g->kev) (void)hipEventDestroy(e);
    if (g->ev0) (void)hipEventDestroy(g->ev0);
    if (g->ev1) (void)hipEventDestroy(g->ev1);
    if (g->stream) (void)hipStreamDestroy(g->stream);
    delete g;
}

// A batched call runs every graph's work on one stream; each graph's own stream is put back
// when the call ends, however it ends.
struct StreamSwap {
    std::vector<std::pair<imin_graph *, hipStream_t>> saved;
    void use(imin_graph *g, hipStream_t s)
    {
        saved.emplace_back(g, g->stream);
        g->stream = s;
    }
    ~StreamSwap()
    {
        for (auto &p : saved) p.first->stream = p.second;
    }
};

// A device buffer of at least `count` elements, kept and grown only when too small.
template <class T>
bool grow(T *&p, size_t &cap, size_t count)
{
    count = std::max<size_t>(count, 1);
    if (p && cap >= count) return true;
    dfree(p);
    cap = 0;
    if (!ok(hipMalloc(&p, count * sizeof(T)))) {
        (void)hipGetLastError();
        return false;
    }
    cap = count;
    return true;
}

struct BatchItem {
    imin_instance *in = nullptr;
    imin_graph *g = nullptr;
    std::vector<int32_t> seeds;
    std::vector<uint32_t> inelig;
    std::vector<uint32_t> cand;  // GreedyReplace: CB
    int32_t rounds = 0;          // greedy rounds at most (GreedyReplace: 2k)
    int32_t nb = 0;              // blocker slots (GreedyReplace: k)
};

// A stream capture that is always ended, and the graph it made, released at scope exit.
struct GraphCapture {
    hipStream_t stream = nullptr;  // non-null while capturing
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int finish()
    {
        hipStream_t s = stream;
        stream = nullptr;
        if (!ok(hipStreamEndCapture(s, &graph)) ||
            !ok(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0))) {
            (void)hipGetLastError();
            return IMIN_EDEVICE;
        }
        return IMIN_OK;
    }
    ~GraphCapture()
    {
        if (stream) {
            hipGraph_t g = nullptr;
            (void)hipStreamEndCapture(stream, &g);
            if (g) (void)hipGraphDestroy(g);
            (void)hipGetLastError();
        }
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
    }
};

}  // namespace host
}  // namespace imin

using namespace imin::host;

extern "C" {

const char *imin_strerror(int status)
{
    switch (status) {
    case IMIN_OK: return "ok";
    case IMIN_EINVAL: return "invalid argument";
    case IMIN_ENOMEM: return "out of memory";
    case IMIN_EDEVICE: return "device error";
    case IMIN_ERANGE: return "size out of range";
    default: return "unknown status";
    }
}

int imin_graph_create(int32_t n, int32_t m, const int32_t *row_ptr, const int32_t *col,
                      const float *prob, imin_graph **out)
{
    return imin_graph_create_model(n, m, row_ptr, col, prob, IMIN_IC, out);
}

int imin_graph_create_model(int32_t n, int32_t m, const int32_t *row_ptr, const int32_t *col,
                            const float *prob, int model, imin_graph **out)
{
    if (!out || !row_ptr || n <= 0 || m < 0) return IMIN_EINVAL;
    if (model != IMIN_IC && model != IMIN_LT) return IMIN_EINVAL;
    if (n == INT32_MAX) return IMIN_ERANGE;
    if (row_ptr[0] != 0 || row_ptr[n] != m) return IMIN_EINVAL;
    for (int32_t v = 0; v < n; ++v)
        if (row_ptr[v + 1] < row_ptr[v]) return IMIN_EINVAL;
    if (m > 0 && (!col || !prob)) return IMIN_EINVAL;
    for (int32_t e = 0; e < m; ++e) {
        if (col[e] < 0 || col[e] >= n) return IMIN_EINVAL;
        if (!(prob[e] >= 0.0f && prob[e] <= 1.0f)) return IMIN_EINVAL;  // rejects NaN
    }
    int ndev = 0;
    if (!ok(hipGetDeviceCount(&ndev)) || ndev <= 0) return IMIN_EDEVICE;

    imin_graph *g = new (std::nothrow) imin_graph();
    if (!g) return IMIN_ENOMEM;
    g->n = n;
    g->m = m;
    if (!ok(hipGetDevice(&g->device))) {
        delete g;
        return IMIN_EDEVICE;
    }
    hipDeviceProp_t prop;
    if (!ok(hipGetDeviceProperties(&prop, g->device))) {
        delete g;
        return IMIN_EDEVICE;
    }
    g->num_cus = std::max(1, prop.multiProcessorCount);
    if (!ok(hipDeviceGetAttribute(&g->clock_khz, hipDeviceAttributeWallClockRate, g->device)) ||
        g->clock_khz <= 0) {
        delete g;
        return IMIN_EDEVICE;
    }
    try {
        g->row_ptr.assign(row_ptr, row_ptr + n + 1);
        g->col.assign(col ? col : row_ptr, col ? col + m : row_ptr);
    } catch (...) {
        delete g;
        return IMIN_ENOMEM;
    }
    const bool lt = model == IMIN_LT;
    const size_t quads = (size_t)std::max<int64_t>(((int64_t)m + 3) / 4, 1);
    const size_t edges = quads * 4;
    // What the host fills lies in one block. Small graphs' arrays lie on the device as they do
    // there and go in one copy: an allocation, a copy or a free costs a graph 10 us each. Larger
    // arrays start where pages of memory do, as allocations of their own would: an 8k-vertex
    // linear-threshold graph's 9,422 samples take 1.08 ms so, and 1.22 packed.
    struct Filled {
        size_t at, words;  // in the block
    };
    size_t staged = 0;
    auto page = [](size_t bytes) {
        return bytes >= (size_t)2 << 20 ? (size_t)2 << 20 : bytes >= (32 << 10) ? (size_t)64 << 10 : 256;
    };
    auto stage = [&](size_t words) {
        const size_t to = std::min<size_t>(page(words * 4), 64 << 10) / 4;
        const size_t at = (staged + to - 1) / to * to;
        staged = at + words;
        return Filled{at, words};
    };
    const Filled f_row = stage((size_t)n + 1), f_col = stage(edges), f_thr = stage(edges);
    const Filled f_in = stage((size_t)n + 1), f_ine = stage((size_t)std::max(m, 1));
    const Filled f_lo = stage(lt ? edges : 0), f_rid = stage((size_t)n), f_vtx = stage((size_t)n);
    const bool one_copy = staged * 4 <= (1 << 20);
    std::vector<uint32_t> host;
    std::vector<int32_t> fill;
    std::vector<uint4> fnode;
    int32_t nclaim = 0, nreach = 0, nsrc = 0;
    imin::ForestShape fshape;
    bool forest = false;
    try {
        host.assign(staged, 0u);  // padding edges have threshold 0: never live
        std::copy(row_ptr, row_ptr + n + 1, host.begin() + f_row.at);
        if (m > 0) std::copy(col, col + m, host.begin() + f_col.at);
        uint32_t *const thr = host.data() + f_thr.at;
        int32_t *const in_ptr = reinterpret_cast<int32_t *>(host.data() + f_in.at);
        int32_t *const in_edge = reinterpret_cast<int32_t *>(host.data() + f_ine.at);
        if (!lt)
            for (int32_t e = 0; e < m; ++e) thr[e] = live_threshold(prob[e]);
        // in-edge index: edge ids grouped by target, ascending (counting sort)
        for (int32_t e = 0; e < m; ++e) ++in_ptr[(size_t)col[e] + 1];
        for (int32_t v = 0; v < n; ++v) in_ptr[(size_t)v + 1] += in_ptr[v];
        fill.assign(in_ptr, in_ptr + n);
        for (int32_t e = 0; e < m; ++e) in_edge[fill[(size_t)col[e]]++] = e;
        // Reach ids: the vertices that need a claim (two or more in-edges), then those with one;
        // the vertices without are numbered below -1.
        int32_t *const rid = reinterpret_cast<int32_t *>(host.data() + f_rid.at);
        int32_t *const vtx = reinterpret_cast<int32_t *>(host.data() + f_vtx.at);
        for (int32_t v = 0; v < n; ++v) {
            const int32_t deg = in_ptr[(size_t)v + 1] - in_ptr[v];
            if (deg > 1) {
                rid[v] = nclaim;
                vtx[nclaim++] = v;
            } else if (deg == 0) {
                rid[v] = -1 - nsrc++;
            }
        }
        nreach = nclaim;
        for (int32_t v = 0; v < n; ++v)
            if (in_ptr[(size_t)v + 1] - in_ptr[v] == 1) {
                rid[v] = nreach;
                vtx[nreach++] = v;
            }
        if (lt) {
            // Linear-threshold model: the in-edges of v split [0, 2^24) into consecutive intervals,
            // edge k of v (ascending id) getting [bound_{k-1}, bound_k) with
            // bound_k = min(2^24, ceil(2^24 * (w_1 + ... + w_k))) from fp64 running sums.
            uint32_t *const lo = host.data() + f_lo.at;
            for (int32_t v = 0; v < n; ++v) {
                double sum = 0.0;
                uint32_t prev = 0;
                for (int32_t k = in_ptr[v]; k < in_ptr[(size_t)v + 1]; ++k) {
                    const int32_t e = in_edge[k];
                    sum += (double)prob[e];
                    const double bound = std::min(16777216.0, std::ceil(sum * 16777216.0));
                    lo[e] = prev;
                    thr[e] = (uint32_t)bound;
                    prev = (uint32_t)bound;
                }
                if (sum > 1.0 + 1e-5) {
                    delete g;
                    return IMIN_EINVAL;
                }
            }
            // Few enough reachable vertices: the in-edges by reach id (launch_forest_index)
            forest = imin::forest_shape(nreach, nsrc, fshape);
            if (forest) {
                fnode.reserve((size_t)nreach);
                uint32_t first = 0;
                for (int32_t r = 0; r < nreach; ++r) {
                    const int32_t v = vtx[r];
                    const uint32_t deg = (uint32_t)(in_ptr[(size_t)v + 1] - in_ptr[v]);
                    fnode.push_back(make_uint4((uint32_t)v, first, deg,
                                               (uint32_t)(row_ptr[(size_t)v + 1] - row_ptr[v])));
                    first += deg;
                }
            }
        }
    } catch (...) {
        delete g;
        return IMIN_ENOMEM;
    }
    g->model = model;
    g->words = (n + 31) / 32;
    g->nclaim = nclaim;
    g->nreach = nreach;
    g->tree = imin::tree_shape(tree_fit(g, 1, false), g->shape);
    g->forest = g->tree && forest;
    g->fshape = fshape;
    g->nsrc = nsrc;
    const size_t records = g->tree ? edges : 0, fedges = g->forest ? (size_t)m : 0;
    auto carve = [&](unsigned char *base) {
        size_t at = one_copy ? (staged * 4 + 255) / 256 * 256 : 0;
        auto take = [&](auto *&p, size_t count) {
            using T = typename std::remove_reference<decltype(*p)>::type;
            const size_t to = page(count * sizeof(T));
            at = (at + to - 1) / to * to;
            p = count > 0 ? reinterpret_cast<T *>(base + at) : nullptr;
            at += count * sizeof(T);
        };
        auto place = [&](auto *&p, Filled f) {
            using T = typename std::remove_reference<decltype(*p)>::type;
            if (one_copy) p = f.words ? reinterpret_cast<T *>(base + f.at * 4) : nullptr;
            else take(p, f.words * 4 / sizeof(T));
        };
        place(g->d_row_ptr, f_row);
        place(g->d_col4, f_col);
        place(g->d_thr_orig, f_thr);
        place(g->d_in_ptr, f_in);
        place(g->d_in_edge, f_ine);
        place(g->d_lo4, f_lo);
        place(g->d_rid_of, f_rid);
        place(g->d_rid_vtx, f_vtx);
        take(g->d_thr4, quads);
        take(g->d_inelig, (size_t)g->words);
        take(g->d_cand, (size_t)g->words);
        take(g->d_seeds, (size_t)n);
        take(g->d_list, (size_t)n);
        take(g->d_D, (size_t)n + (size_t)nreach);
        take(g->d_stats, (size_t)kCallStats);
        take(g->d_ctrl, (size_t)imin::kCtrlWords);
        take(g->d_sctrl, (size_t)3);
        take(g->d_inst, (size_t)1);
        take(g->d_part_d, (size_t)g->parts);
        take(g->d_part_i, (size_t)g->parts);
        take(g->d_x, (size_t)1);
        take(g->d_tl, lt ? 2 * quads : 0);
        take(g->d_edge, lt ? 0 : edges);
        take(g->d_tedge, records);
        take(g->d_code, lt ? 0 : records / 4);
        take(g->d_fnode, fedges ? (size_t)nreach : 0);
        take(g->d_fin16, fedges);
        take(g->d_fbound, fedges);
        take(g->d_fsrc, fedges);
        return at;
    };
    if (!ok(hipStreamCreateWithFlags(&g->stream, hipStreamNonBlocking)) ||
        !ok(hipEventCreate(&g->ev0)) || !ok(hipEventCreate(&g->ev1)) ||
        !ok(hipMalloc(&g->block, carve(nullptr)))) {
        (void)hipGetLastError();
        g->block = nullptr;
        destroy(g);
        return IMIN_ENOMEM;
    }
    carve(g->block);
    const uint32_t *const orig = reinterpret_cast<const uint32_t *>(g->d_thr_orig);
    const uint32_t *const targets = reinterpret_cast<const uint32_t *>(g->d_col4);
    auto send = [&](void *to, Filled f) {
        return f.words == 0 ||
               ok(hipMemcpy(to, host.data() + f.at, f.words * 4, hipMemcpyHostToDevice));
    };
    const bool sent = one_copy
                          ? send(g->block, Filled{0, staged})
                          : send(g->d_row_ptr, f_row) && send(g->d_col4, f_col) &&
                                send(g->d_thr_orig, f_thr) && send(g->d_in_ptr, f_in) &&
                                send(g->d_in_edge, f_ine) && send(g->d_lo4, f_lo) &&
                                send(g->d_rid_of, f_rid) && send(g->d_rid_vtx, f_vtx);
    if (!sent ||
        (g->forest && !ok(hipMemcpy(g->d_fnode, fnode.data(), fnode.size() * sizeof(uint4),
                                    hipMemcpyHostToDevice))) ||
        !ok(imin::launch_edge_records(targets, g->d_row_ptr, g->d_rid_of, orig,
                                      reinterpret_cast<const uint32_t *>(g->d_lo4), m, (int64_t)edges,
                                      g->d_tedge, reinterpret_cast<uint8_t *>(g->d_code), g->d_edge,
                                      reinterpret_cast<uint32_t *>(g->d_thr4),
                                      reinterpret_cast<uint32_t *>(g->d_tl), g->stream)) ||
        (g->forest &&
         !ok(imin::launch_forest_index(g->d_in_ptr, g->d_in_edge, targets, g->d_row_ptr, n, m,
                                       g->d_rid_of, orig, g->d_fnode, g->d_fin16, g->d_fbound,
                                       g->d_fsrc, g->stream))) ||
        !ok(hipStreamSynchronize(g->stream))) {
        destroy(g);
        return IMIN_EDEVICE;
    }
    *out = g;
    return IMIN_OK;
}

void imin_graph_destroy(imin_graph *g) { destroy(g); }

int imin_set_launch(imin_graph *g, int32_t slots, int64_t extra_cap)
{
    if (!g || slots < 0 || extra_cap < 0) return IMIN_EINVAL;
    if (slots > IMIN_MAX_SLOTS) return IMIN_ERANGE;
    g->force_slots = slots;
    g->force_xcap = extra_cap;
    return IMIN_OK;
}

}  // extern "C"

namespace {

// One Algorithm 2 call (counts != NULL) or a reachability-only estimate (counts == NULL).
int one_call(imin_graph *g, const int32_t *S, int32_t nS, const uint8_t *blocked,
             uint32_t theta, uint64_t seed, uint64_t *counts, imin_stats *stats,
             int32_t *n_seeds)
{
    if (!g || theta == 0) return IMIN_EINVAL;
    if (theta > kMaxTheta) return IMIN_ERANGE;
    const bool reach_only = counts == nullptr;
    std::vector<int32_t> seeds;
    std::vector<uint32_t> inelig;
    int rc = seed_setup(g, S, nS, seeds, inelig);
    if (rc) return rc;
    if (blocked) {
        for (int32_t v = 0; v < g->n; ++v) {
            if (!blocked[v]) continue;
            // a seed cannot be blocked (Definition 2: B is a subset of V \ S)
            if (std::binary_search(seeds.begin(), seeds.end(), v)) return IMIN_EINVAL;
            inelig[v >> 5] |= 1u << (v & 31);
        }
    }
    rc = begin_call(g, seeds);
    if (rc) return rc;
    rc = prepare_workspaces(g, theta, reach_only);
    if (rc) return rc;
    rc = ensure_ovf(g, theta);
    if (rc) return rc;
    rc = ensure_sj(g, theta);
    if (rc) return rc;
    rc = upload_call_state(g, seeds, inelig, nullptr, seed, theta, 0, !reach_only);
    if (rc) return rc;
    if (g->wave_first) g->auto_pending = false;  // no later round to judge the first one for
    rc = decrease_round(g, (int32_t)seeds.size(), theta, seed, 0, reach_only);
    if (rc) return rc;
    const bool pinned = pinned_counts(g);
    std::vector<unsigned long long> D;
    if (!reach_only && !pinned) {
        D.resize((size_t)g->n);
        if (!ok(hipMemcpyAsync(D.data(), g->d_D, (size_t)g->n * sizeof(unsigned long long),
                               hipMemcpyDeviceToHost, g->stream)))
            return IMIN_EDEVICE;
    }
    imin_stats st;
    rc = finish_call(g, &st, !reach_only && pinned ? g->d_D : nullptr, true);
    if (rc) return rc;
    end_masks(g, {});
    if (!reach_only)
        std::memcpy(counts, pinned ? g->at.D : D.data(), (size_t)g->n * sizeof(uint64_t));
    if (stats) *stats = st;
    *n_seeds = (int32_t)seeds.size();
    return IMIN_OK;
}

}  // namespace

extern "C" {

int imin_decrease(imin_graph *g, const int32_t *S, int32_t nS, const uint8_t *blocked,
                  uint32_t theta, uint64_t seed, uint64_t *counts, imin_stats *stats)
{
    if (!counts) return IMIN_EINVAL;
    int32_t ns = 0;
    return one_call(g, S, nS, blocked, theta, seed, counts, stats, &ns);
}

int imin_spread(imin_graph *g, const int32_t *S, int32_t nS, const uint8_t *blocked,
                uint32_t theta, uint64_t seed, double *spread, imin_stats *stats)
{
    if (!spread) return IMIN_EINVAL;
    imin_stats st;
    int32_t ns = 0;
    const int rc = one_call(g, S, nS, blocked, theta, seed, nullptr, &st, &ns);
    if (rc) return rc;
    *spread = (double)ns + (double)st.reached / (double)theta;
    if (stats) *stats = st;
    return IMIN_OK;
}

int imin_greedy(imin_graph *g, const int32_t *S, int32_t nS, int32_t b, uint32_t theta,
                uint64_t seed, int mode, int32_t *blockers, int32_t *n_blockers,
                imin_stats *stats)
{
    if (!g || theta == 0 || b < 0 || !n_blockers || (b > 0 && !blockers)) return IMIN_EINVAL;
    if (mode != IMIN_AG && mode != IMIN_GR) return IMIN_EINVAL;
    if (theta > kMaxTheta) return IMIN_ERANGE;
    std::vector<int32_t> seeds;
    std::vector<uint32_t> inelig;
    int rc = seed_setup(g, S, nS, seeds, inelig);
    if (rc) return rc;
    const int32_t ns = (int32_t)seeds.size();
    rc = begin_call(g, seeds);
    if (rc) return rc;
    rc = prepare_workspaces(g, theta);
    if (rc) return rc;
    rc = ensure_ovf(g, theta);
    if (rc) return rc;
    rc = ensure_sj(g, theta);
    if (rc) return rc;
    // AG: the rounds; GR: the out-neighbours of the merged seed, seeds excluded (Algorithm 4), and
    // its first phase's rounds.
    std::vector<uint32_t> cand;
    const int32_t most = mode == IMIN_AG ? g->n - ns : gr_candidates(g, seeds, inelig, cand);
    const int32_t rounds = std::min(b, most);
    rc = upload_call_state(g, seeds, inelig, mode == IMIN_GR ? &cand : nullptr, seed, theta, rounds,
                           false);
    if (rc) return rc;
    // the kernels write the blockers, and the last one chosen, into the pinned block
    const imin::host::CallPin &at = g->at;

    std::vector<int32_t> B;
    uint64_t call = 0;
    if (mode == IMIN_AG) {
        for (int32_t r = 0; r < rounds; ++r) {
            rc = decrease_round(g, ns, theta, seed, call);
            if (rc) return rc;
            ++call;
            if (!ok(imin::launch_argmax_apply(g->d_D, g->d_inelig, 0, g->n, g->d_part_d,
                                              g->d_part_i, g->parts, g->d_inelig, nullptr,
                                              at.B, r, at.x, thr_w(g), g->mask_rec(),
                                              g->d_in_ptr, g->d_in_edge, clock_of(g), g->stream)))
                return IMIN_EDEVICE;
            if (rounds >= 4 && (rc = fit_rounds(g, r, theta))) return rc;
        }
    } else {
        const int32_t k = rounds;
        for (int32_t r = 0; r < k; ++r) {
            rc = decrease_round(g, ns, theta, seed, call);
            if (rc) return rc;
            ++call;
            if (!ok(imin::launch_argmax_apply(g->d_D, g->d_cand, 1, g->n, g->d_part_d,
                                              g->d_part_i, g->parts, g->d_inelig, g->d_cand,
                                              at.B, r, at.x, thr_w(g), g->mask_rec(),
                                              g->d_in_ptr, g->d_in_edge, clock_of(g), g->stream)))
                return IMIN_EDEVICE;
            if (k >= 3 && (rc = fit_rounds(g, r, theta))) return rc;
        }
        if (k > 0 && !ok(hipStreamSynchronize(g->stream))) return IMIN_EDEVICE;
        B.assign(at.B, at.B + k);
        for (int32_t v : B)
            if (v < 0) return IMIN_EDEVICE;
        const std::vector<int32_t> snapshot = B;
        for (int32_t i = k - 1; i >= 0; --i) {
            const int32_t u = snapshot[(size_t)i];
            const int32_t slot =
                (int32_t)(std::find(B.begin(), B.end(), u) - B.begin());
            rc = decrease_round(g, ns, theta, seed, call, false, u);
            if (rc) return rc;
            ++call;
            if (!ok(imin::launch_argmax_apply(g->d_D, g->d_inelig, 0, g->n, g->d_part_d,
                                              g->d_part_i, g->parts, g->d_inelig, nullptr,
                                              at.B, slot, at.x, thr_w(g), g->mask_rec(),
                                              g->d_in_ptr, g->d_in_edge, clock_of(g), g->stream)) ||
                !ok(hipStreamSynchronize(g->stream)))
                return IMIN_EDEVICE;
            const int32_t x = *at.x;
            if (x < 0) return IMIN_EDEVICE;
            B[(size_t)slot] = x;
            if (x == u) break;
        }
    }
    imin_stats st;
    rc = finish_call(g, &st, nullptr, false);
    if (rc) return rc;
    if (mode == IMIN_AG) B.assign(at.B, at.B + rounds);
    for (int32_t v : B)
        if (v < 0) return IMIN_EDEVICE;
    end_masks(g, B);
    std::copy(B.begin(), B.end(), blockers);
    *n_blockers = (int32_t)B.size();
    if (stats) *stats = st;
    return IMIN_OK;
}

int imin_set_small(imin_graph *g, int32_t enable, const imin_launch *launch)
{
    if (!g || enable < -1 || enable > 1 || !launch_ok(launch)) return IMIN_EINVAL;
    g->small_mode = enable;
    g->small_auto_off = false;
    g->small_launch = launch ? *launch : imin_launch{0, 0, 0, 0, 0};
    return IMIN_OK;
}

int imin_set_workgroup(imin_graph *g, int32_t threads)
{
    if (!g || (threads != -1 && threads != 0 && threads != 64 && threads != 128 &&
               threads != 256 && threads != 512 && threads != 1024))
        return IMIN_EINVAL;
    imin::TreeFit fit = tree_fit(g, 1, false);
    fit.block = threads;
    imin::TreeShape s;
    if (threads > 0 && (!g->tree || !imin::tree_shape(fit, s))) return IMIN_ERANGE;
    g->force_block = threads;
    return IMIN_OK;
}

int imin_greedy_batch(imin_instance *inst, int32_t count, int mode, const imin_launch *launch)
{
    if (!inst || count <= 0 || (mode != IMIN_AG && mode != IMIN_GR) || !launch_ok(launch))
        return IMIN_EINVAL;
    const bool gr = mode == IMIN_GR;
    const imin_launch shape = launch ? *launch : imin_launch{0, 0, 0, 0, 0};
    std::vector<BatchItem> items((size_t)count);
    std::vector<imin_graph *> graphs;
    uint64_t theta_sum = 0;
    for (int32_t i = 0; i < count; ++i) {
        imin_instance &in = inst[i];
        if (!in.g || in.theta == 0 || in.b < 0 || !in.n_blockers || (in.b > 0 && !in.blockers))
            return IMIN_EINVAL;
        if (in.g->device != inst[0].g->device || in.g->model != inst[0].g->model)
            return IMIN_EINVAL;
        BatchItem &it = items[(size_t)i];
        it.in = &in;
        it.g = in.g;
        int rc = seed_setup(in.g, in.S, in.nS, it.seeds, it.inelig);
        if (rc) return rc;
        if (gr) {
            const int32_t k = std::min(gr_candidates(in.g, it.seeds, it.inelig, it.cand), in.b);
            it.nb = k;
            it.rounds = 2 * k;
        } else {
            it.rounds = std::min<int32_t>(in.b, in.g->n - (int32_t)it.seeds.size());
            it.nb = it.rounds;
        }
        theta_sum += in.theta;
        graphs.push_back(in.g);
    }
    std::sort(graphs.begin(), graphs.end());
    if (std::adjacent_find(graphs.begin(), graphs.end()) != graphs.end()) return IMIN_EINVAL;
    if (theta_sum > kMaxTheta) return IMIN_ERANGE;
    // Instances with more rounds first: the ones still active in round r form a prefix.
    std::stable_sort(items.begin(), items.end(),
                     [](const BatchItem &a, const BatchItem &b) { return a.rounds > b.rounds; });
    if (!ok(hipSetDevice(inst[0].g->device))) return IMIN_EDEVICE;
    for (imin_graph *g : graphs)
        if (!ok(hipStreamSynchronize(g->stream))) return IMIN_EDEVICE;
    const hipStream_t bs = inst[0].g->stream;
    StreamSwap swap;
    for (imin_graph *g : graphs) swap.use(g, bs);

    imin_graph *g0 = inst[0].g;
    g0->kev_used = 0;
    if (!ok(hipEventRecord(g0->ev0, bs))) return IMIN_EDEVICE;
    // Call state of every instance, staged in one buffer and put in place by one kernel.
    std::vector<imin::InstanceDesc> table((size_t)count);
    std::vector<imin::BatchStage> stages((size_t)count);
    std::vector<int32_t> stage, rounds((size_t)count);
    std::vector<uint32_t> prefix((size_t)count + 1, 0u);
    int32_t max_rounds = 0, max_nb = 0, gr_runs = 0;
    for (int32_t i = 0; i < count; ++i) {
        BatchItem &it = items[(size_t)i];
        imin_graph *g = it.g;
        const int rc = ensure_B(g, it.nb);
        if (rc) return rc;
        describe(g, (int32_t)it.seeds.size(), it.in->seed, it.in->theta);
        table[(size_t)i] = g->h_inst;
        table[(size_t)i].sample_base = prefix[(size_t)i];
        table[(size_t)i].gr_k = gr ? it.nb : -1;
        prefix[(size_t)i + 1] = prefix[(size_t)i] + it.in->theta;
        rounds[(size_t)i] = it.nb;  // blocker slots gathered at the end
        max_rounds = std::max(max_rounds, it.rounds);
        max_nb = std::max(max_nb, it.nb);
        if (gr && it.nb > 0) ++gr_runs;
        imin::BatchStage &S = stages[(size_t)i];
        S.seeds = (int64_t)stage.size();
        stage.insert(stage.end(), it.seeds.begin(), it.seeds.end());
        S.bits = (int64_t)stage.size();
        S.words = (int32_t)it.inelig.size();
        for (uint32_t w : it.inelig) stage.push_back((int32_t)w);
        S.prev = (int64_t)stage.size();
        S.nprev = g->mask_known ? (int32_t)g->masked.size() : -1;
        if (g->mask_known) stage.insert(stage.end(), g->masked.begin(), g->masked.end());
        g->mask_known = false;
        g->masked.clear();
        append_set_bits(it.inelig, g->masked);
        S.now = (int64_t)stage.size();
        S.nnow = (int32_t)g->masked.size();
        stage.insert(stage.end(), g->masked.begin(), g->masked.end());
        S.cand = -1;
        if (gr) {
            S.cand = (int64_t)stage.size();
            for (uint32_t w : it.cand) stage.push_back((int32_t)w);
        }
    }
    const int32_t stride = imin::kGatherB + std::max(max_nb, 1);
    MultiSize size;
    for (const BatchItem &it : items) size.add(it.g);
    // The batch's scratch stays with its first graph for the next batch that graph leads
    // (same shape: nothing is allocated or cleared again).
    if (!g0->batch_ms) {
        g0->batch_ms = new (std::nothrow) MultiScratch();
        if (!g0->batch_ms) return IMIN_ENOMEM;
    }
    MultiScratch &ms = *g0->batch_ms;
    int rc = multi_alloc(ms, g0->num_cus, size, prefix[(size_t)count], count, bs);
    if (rc) {
        multi_free(ms);
        return rc;
    }
    if (!grow(ms.table, ms.table_cap, (size_t)count) ||
        !grow(ms.stages, ms.stages_cap, (size_t)count) ||
        !grow(ms.stage, ms.stage_cap, stage.size()) ||
        !grow(ms.rounds, ms.rounds_cap, (size_t)count) ||
        !grow(ms.out, ms.out_cap, (size_t)count * stride))
        return IMIN_ENOMEM;
    if (!ok(hipMemcpyAsync(ms.table, table.data(), table.size() * sizeof(imin::InstanceDesc),
                           hipMemcpyHostToDevice, bs)) ||
        !ok(hipMemcpyAsync(ms.stages, stages.data(), stages.size() * sizeof(imin::BatchStage),
                           hipMemcpyHostToDevice, bs)) ||
        !ok(hipMemcpyAsync(ms.stage, stage.data(), stage.size() * sizeof(int32_t),
                           hipMemcpyHostToDevice, bs)) ||
        !ok(hipMemcpyAsync(ms.rounds, rounds.data(), rounds.size() * sizeof(int32_t),
                           hipMemcpyHostToDevice, bs)) ||
        !ok(imin::launch_batch_setup(ms.table, ms.stages, ms.stage, count, bs)))
        return IMIN_EDEVICE;
    // Rounds: every launch is queued at once; nothing waits for the host until the end
    // (GreedyReplace: one word read back per round, the count of runs that have ended).
    const bool lt = g0->model == IMIN_LT;
    if (!ok(imin::launch_fill_u32(ms.ctrl + 9, 1, 0, bs))) return IMIN_EDEVICE;
    if (shape.graph && !gr) {
        // One HIP graph of kernel nodes for all rounds (slots clear their own maps when
        // their epochs wrap, so no memset is ever needed inside). Every kernel reads the
        // call's state through the device table, so the graph depends only on the launch
        // structure below; a call with the same structure replays the kept graph.
        std::vector<int64_t> key = {count, max_rounds, lt ? 1 : 0, g0->num_cus,
                                    shape.waves_per_cu, shape.quad_limit, shape.pick_div,
                                    shape.pack_per_cu, (int64_t)(uintptr_t)ms.table,
                                    (int64_t)(uintptr_t)ms.ctrl, (int64_t)(uintptr_t)ms.pi,
                                    (int64_t)(uintptr_t)ms.si, (int64_t)(uintptr_t)ms.oi,
                                    (int64_t)(uintptr_t)ms.part_d, (int64_t)ms.cap,
                                    (int64_t)(uintptr_t)ms.main_ws.map, ms.main_ws.slots,
                                    ms.main_ws.n, ms.main_ws.lcap, ms.main_ws.xcap,
                                    (int64_t)(uintptr_t)ms.big_ws.map, ms.big_ws.slots,
                                    ms.tree ? 1 : 0, ms.forest ? 1 : 0, ms.split ? 1 : 0,
                                    (int64_t)(uintptr_t)ms.main_tw.base, ms.main_tw.slots,
                                    ms.main_tw.lcap, ms.main_tw.xcap, ms.main_tw.nclaim,
                                    (int64_t)(uintptr_t)ms.big_tw.base, ms.big_tw.xcap,
                                    ms.shape.block, (int64_t)ms.shape.lds,
                                    (int64_t)(uintptr_t)ms.leaf, (int64_t)(uintptr_t)ms.fws.base,
                                    ms.fws.entries, ms.fshape.block, ms.fws.slots,
                                    (int64_t)(uintptr_t)ms.low_ws.base, ms.low_ws.entries,
                                    ms.low_ws.slots, (int64_t)ms.low_shape.lds,
                                    (int64_t)ms.fshape.lds};
        {
            int32_t act = count;
            for (int32_t r = 0; r < max_rounds; ++r) {
                while (act > 0 && items[(size_t)act - 1].rounds <= r) --act;
                key.push_back(act);
                key.push_back(prefix[(size_t)act]);
            }
        }
        if (!ms.exec || ms.exec_key != key) {
            if (ms.exec) (void)hipGraphExecDestroy(ms.exec);
            ms.exec = nullptr;
            ms.exec_key.clear();
            GraphCapture cap;
            if (!ok(hipStreamBeginCapture(bs, hipStreamCaptureModeThreadLocal)))
                return IMIN_EDEVICE;
            cap.stream = bs;
            int32_t act = count;
            for (int32_t r = 0; r < max_rounds; ++r) {
                while (act > 0 && items[(size_t)act - 1].rounds <= r) --act;
                rc = multi_round(ms, ms.table, act, prefix[(size_t)act], (uint32_t)r, shape,
                                 g0->num_cus, true, false, lt, bs);
                if (rc) return rc;
            }
            rc = cap.finish();
            if (rc) return rc;
            ms.exec = cap.exec;  // kept with the scratch
            cap.exec = nullptr;
            ms.exec_key = std::move(key);
        }
        hipEvent_t k0, k1;
        rc = kernel_events(g0, &k0, &k1);
        if (rc) return rc;
        if (!ok(hipEventRecord(k0, bs)) || !ok(hipGraphLaunch(ms.exec, bs)) ||
            !ok(hipEventRecord(k1, bs)))
            return IMIN_EDEVICE;
    } else {
        int32_t active = count;
        for (int32_t r = 0; r < max_rounds; ++r) {
            while (active > 0 && items[(size_t)active - 1].rounds <= r) --active;
            hipEvent_t k0, k1;
            rc = kernel_events(g0, &k0, &k1);
            if (rc) return rc;
            if (!ok(hipEventRecord(k0, bs))) return IMIN_EDEVICE;
            rc = multi_round(ms, ms.table, active, prefix[(size_t)active], (uint32_t)r,
                             shape, g0->num_cus, true, gr, lt, bs);
            if (rc) return rc;
            if (!ok(hipEventRecord(k1, bs))) return IMIN_EDEVICE;
            if (gr) {
                // every replacement pass that can still run has stopped: no more rounds
                uint32_t ended = 0;
                if (!ok(hipMemcpyAsync(&ended, ms.ctrl + 9, sizeof(ended), hipMemcpyDeviceToHost,
                                       bs)) ||
                    !ok(hipStreamSynchronize(bs)))
                    return IMIN_EDEVICE;
                if ((int32_t)ended >= gr_runs) break;
            }
        }
    }
    // Results: every graph's blocker slots, counters and error flag, gathered into one
    // buffer, then one copy and one wait.
    std::vector<int32_t> out((size_t)count * stride);
    if (!ok(imin::launch_batch_gather(ms.table, ms.rounds, ms.out, stride, count, bs)) ||
        !ok(hipMemcpyAsync(out.data(), ms.out, out.size() * sizeof(int32_t),
                           hipMemcpyDeviceToHost, bs)) ||
        !ok(hipEventRecord(g0->ev1, bs)) || !ok(hipEventSynchronize(g0->ev1)))
        return IMIN_EDEVICE;
    uint32_t wave_err = 0, wg_err = 0;
    rc = multi_errors(ms, &wave_err, &wg_err, bs);
    if (rc) return rc;
    if (wave_err || wg_err) return IMIN_EDEVICE;
    std::vector<std::vector<int32_t>> B((size_t)count);
    std::vector<std::array<unsigned long long, kStats>> st((size_t)count);
    std::vector<uint32_t> err((size_t)count);
    for (int32_t i = 0; i < count; ++i) {
        const int32_t *o = out.data() + (size_t)i * stride;
        for (int k = 0; k < kStats; ++k)
            st[(size_t)i][k] = (unsigned long long)(uint32_t)o[2 * k] |
                               ((unsigned long long)(uint32_t)o[2 * k + 1] << 32);
        err[(size_t)i] = (uint32_t)o[imin::kGatherErr];
        B[(size_t)i].assign(o + imin::kGatherB, o + imin::kGatherB + items[(size_t)i].nb);
    }
    float total_ms = 0.0f;
    if (!ok(hipEventElapsedTime(&total_ms, g0->ev0, g0->ev1))) return IMIN_EDEVICE;
    double kms = 0.0;
    for (size_t k = 0; k + 1 < g0->kev_used; k += 2) {
        float x = 0.0f;
        if (!ok(hipEventElapsedTime(&x, g0->kev[k], g0->kev[k + 1]))) return IMIN_EDEVICE;
        kms += x;
    }
    for (int32_t i = 0; i < count; ++i) {
        if (err[(size_t)i] != 0) return IMIN_EDEVICE;
        for (int32_t v : B[(size_t)i])
            if (v < 0) return IMIN_EDEVICE;
    }
    for (int32_t i = 0; i < count; ++i) {
        BatchItem &it = items[(size_t)i];
        end_masks(it.g, B[(size_t)i]);
        std::copy(B[(size_t)i].begin(), B[(size_t)i].end(), it.in->blockers);
        *it.in->n_blockers = it.nb;
        if (it.in->stats) {
            imin_stats &o = *it.in->stats;
            o.samples = st[(size_t)i][0];
            o.reached = st[(size_t)i][1];
            o.edges_scanned = st[(size_t)i][2];
            o.live_edges = st[(size_t)i][3];
            o.spilled = st[(size_t)i][4];
            o.wave_samples = st[(size_t)i][5];
            o.pack_samples = st[(size_t)i][6];
            o.device_ms = total_ms;
            o.kernel_ms = kms;
        }
    }
    return IMIN_OK;
}

}  // extern "C"
