// tree.hip -- Algorithm 2 of arXiv 2302.13529 on gfx950, one workgroup per sample, with every
// claim made in LDS.
//
// What bounds it. Measured on MI355X, random accesses of 64-lane waves: 32- and 64-bit atomics
// on global memory run at 17-28 G lanes/s whatever level of the memory holds the line (17.5
// over 17 GB, 27 inside L2); loads that miss L2 at 49 G lines/s from HBM and 55 from the
// memory-side cache, a limit that 150 lines in flight per compute unit already reach; L2 hits
// at hundreds of G. So the kernel keeps atomics off global memory wherever a sample's size
// multiplies them, and then counts lines:
//   * claims. A vertex needs a claim only when it has two or more in-edges; those vertices
//     are numbered densely (reach ids below nclaim), and the sample's visited set is a bitmap
//     of nclaim bits in LDS (141 KB of 160 for a 4M-vertex R-MAT graph with 35M edges). A
//     vertex with one in-edge can only be reached through it. Under the linear-threshold
//     model (Section V-E) every vertex has at most one live in-edge, so nothing is ever
//     claimed twice and there is no bitmap at all;
//   * thresholds. The first test of a coin reads a byte per edge (threshold_code); only the
//     edges that pass, about 6 % more than are live, cost a 16-byte record, which holds the
//     exact threshold, the target's reach id and its row range;
//   * order. A wave's live edges pass through an LDS queue in frontier order, so a batch of 64
//     is claimed with every lane at work, a parent's children get consecutive local ids and
//     the local arrays are written in full lines. Waves take chunks of the frontier and need
//     no barrier until the level ends;
//   * subtree sizes. With consecutive children, sizes are summed over runs of equal parents
//     inside a wave; only runs that may go on elsewhere and the few vertices whose dominator
//     is not their BFS parent use atomics;
//   * counts. A reached vertex's own 1 goes into bit-sliced per-slot counters, one pass over
//     the bitmap per sample; only subtree sizes above 1 are added into D with atomics.
// Against the kernel of decrease.hip (a 64-bit global atomic per claim): 5000 samples of that
// R-MAT graph, 370k vertices each, 277 -> 167 ms (L2 misses per reached vertex 7.1 -> 3.1);
// 10,000 samples of a 131k-vertex one 17.3 -> 8.3 ms; linear threshold, 1000 samples of a
// 1M-vertex one, 298k vertices each, 53 -> 36 ms.
//
// The dominator tree (Section V-B3) comes from raising the BFS tree: t(v) <- NCA_t of t(v) and
// v's reached predecessors, in place and in any order, until a whole pass changes nothing.
// Why unordered, unsynchronised passes are right: (1) every value t(v) ever holds is dominated
// by (or is) each strict dominator d of v. A walk from a predecessor of v never passes such a
// d without standing on it, because a strict dominator of a vertex x is on or above every
// value t(x) ever held; and of two walkers, one on d and one below, the one below moves (its
// BFS index is larger). So the NCA found, and hence the new t(v), is on or below d too. (2) A
// pass that stores anything for v stores only values above the one it read, so t(v) is strictly
// higher after it, and passes end. (3) In a pass without a store the tree stood still: t(v) is
// an ancestor of every predecessor of v, the tree paths are a post-fixpoint of the dominator
// equations, and by (1) they hold every dominator: the tree is the dominator tree.
#include "imin_internal.h"
#include "philox.h"
#include "planes.h"
#include "wave.h"

#include <algorithm>
#include <cstddef>

namespace imin {
namespace {

using namespace wave;
using namespace planes;

constexpr int kItems = 2;        // items in flight per lane
constexpr int kRing = 128;       // a wave's queue of live edges: at most 63 wait for company
constexpr int kHeavy = 128;      // a row of more items is shared by all waves,
constexpr int kPart = 256;       // in parts of that many
constexpr int kHeavyCap = 256;

// LDS of a workgroup of B threads ahead of its bitmap.
template <int B>
struct TreeHead {
    // one set of level counters in use, one being cleared, one being read (by level mod 3)
    int chunk[3];     // next chunk of the level's frontier
    int grown[3];     // vertices the level has claimed
    int nheavy[3];
    uint32_t idx;
    int nextra;
    int changed;
    // behind here: the BFS; with the bitmap, free after it
    int heavy[3][B > 64 ? kHeavyCap : 1];  // row start, row end, source
    uint32_t qe[B / 64][kRing];       // live edge
    int qs[B / 64][kRing];            // its source's local id
    uint8_t mark[B / 64][64 * kItems];        // a wave's round: the rows that begin at its items
};

template <int B>
__host__ __device__ constexpr size_t head_bytes()
{
    return (sizeof(TreeHead<B>) + 15) / 16 * 16;
}

// Bytes of the head that hold no per-sample scalars: reused by the dominator steps.
template <int B>
__host__ __device__ constexpr size_t free_offset()
{
    return offsetof(TreeHead<B>, heavy);
}

struct TreeCall {
    const int32_t *row_ptr;
    const uint4 *edge;
    const uint32_t *code;
    const uint4 *thr4;
    const uint4 *tl;
    const int32_t *seeds;
    const int32_t *rid_vtx;
    int32_t nseeds;
    int32_t nclaim, nreach;
    uint32_t key_lo, key_hi;
    unsigned long long *D;
    unsigned long long *stats;
    int32_t own_thr;  // the exact thresholds are thr4's, not the records' (a query's masks)
};

// Thresholds in a byte. A coin below a threshold t has a value of at most t - 1, and so has its
// code: the exponent and the three leading mantissa bits of the value as a float, which grow
// with it. An edge whose coin passes this test (about 6 % more than are live) is decided by
// the exact threshold in its record. Rows are 21 edges long on average where it matters, so
// the byte array is a quarter of the lines, and a level's hub rows stay in L2.
__device__ __forceinline__ int coin_code(uint32_t coin)
{
    return (int)(__float_as_uint((float)coin) >> 20) - 1015;
}

__device__ __forceinline__ uint32_t threshold_code(uint32_t thr)
{
    return thr == 0u ? 0u : (uint32_t)max(1, coin_code(thr - 1u));
}

struct TreeSlot {
    int2 *rng;
    int32_t *dom, *rid, *par, *acc, *lvl, *lid;
    int4 *extra;
    uint32_t *planes;
};

// A wave-uniform value in scalar registers.
template <class T>
__device__ __forceinline__ T scalar(T v)
{
    if constexpr (sizeof(T) == 4) {
        return (T)__builtin_amdgcn_readfirstlane((int)v);
    } else {
        const unsigned long long x = (unsigned long long)v;
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
        return (T)(((unsigned long long)hi << 32) | lo);
    }
}

template <class T>
__device__ __forceinline__ T ld(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <class T>
__device__ __forceinline__ void st(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Nearest common ancestor of x and y in the tree t (larger index walks up). Vertices below
// `deep` are children of the root: a walk that gets there needs no more loads.
template <class T>
__device__ __forceinline__ int tree_nca(const T *t, int deep, int x, int y)
{
    while (x != y) {
        if (x > y) x = x < deep ? 0 : (int)ld(&t[x]);
        else y = y < deep ? 0 : (int)ld(&t[y]);
    }
    return x;
}

// Inclusive running maximum of non-negative values across the wave, as wave_scan.
__device__ __forceinline__ int wave_scan_max(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));
    return v;
}

// A wave's queue of live edges, in frontier order: a ring in LDS.
struct WaveQueue {
    uint32_t *qe;
    int *qs;
    int head, n;  // uniform
};

// A queued edge's record, and whether it is live: an edge queued under the independent cascade
// has passed the test of the codes and is decided here.
template <bool kLT>
__device__ __forceinline__ bool follow(const TreeCall &c, const WaveQueue &q, bool has, uint32_t j,
                                       uint4 &r, int &from)
{
    r = make_uint4(0, 0, 0, 0);
    from = 0;
    uint32_t e = 0;
    if (has) {
        const int at = (q.head + lane_id()) & (kRing - 1);
        e = q.qe[at];
        r = glob(c.edge)[e];
        from = q.qs[at];
        if (!kLT && c.own_thr) r.w = reinterpret_cast<const uint32_t *>(glob(c.thr4))[e];
    }
    if (kLT) return has;
    uint32_t k0 = c.key_lo, k1 = c.key_hi, w0, w1, w2, w3;
    asm volatile("" : "+s"(k0), "+s"(k1));
    philox4x32_10(e >> 2, j, k0, k1, w0, w1, w2, w3);
    const uint32_t w = (e & 2) ? ((e & 1) ? w3 : w2) : ((e & 1) ? w1 : w0);
    return has && (w >> 8) < r.w;
}

// Where the live edges of a workgroup's sample go.
template <bool kLT>
struct GroupSink {
    const TreeCall &c;
    const TreeSlot &sv;
    int64_t xcap;
    bool reach_only;
    uint32_t *bm;
    int *nextra;
    int base;      // local id of the level's first claim
    int *grown;
    bool shared;   // the rows at hand are shared with other waves

    __device__ __forceinline__ bool full() const { return false; }

    // The first k (at most 64) queued edges: claim their targets. The winners get consecutive
    // local ids in queue order, so equal parents are adjacent; a run of equal parents that may
    // go on in another batch (the first, the last, any of a shared row) is marked (sign of
    // acc).
    __device__ __forceinline__ void consume(WaveQueue &q, int k, uint32_t j, uint32_t &live)
    {
        const int lane = lane_id();
        uint4 r;
        int from;
        const bool has = follow<kLT>(c, q, lane < k, j, r, from);
        live += has ? 1u : 0u;
        bool won = has;
        if (!kLT && has && r.z < (uint32_t)c.nclaim) {
            const uint32_t bit = 1u << (r.z & 31);
            won = (atomicOr(&bm[r.z >> 5], bit) & bit) == 0u;
            // another live edge into a reached vertex; edges from the merged seed never matter
            // for dominators (their targets are its children)
            if (!won && from != 0 && !reach_only) {
                const int x = atomicAdd(nextra, 1);
                if (x < xcap) sv.extra[x] = make_int4(from, (int)r.z, 0, 0);
            }
        }
        const unsigned long long b = __ballot(won);
        if (b) {
            const int wins = __builtin_popcountll(b);
            int first = 0;
            if (lane == 0) first = atomicAdd(grown, wins);
            first = base + __builtin_amdgcn_readfirstlane(first);
            const int id = first + __builtin_popcountll(b & ((1ull << lane) - 1ull));
            const int p0 = __builtin_amdgcn_readlane(from, __builtin_ctzll(b));
            const int p1 = __builtin_amdgcn_readlane(from, 63 - __builtin_clzll(b));
            if (won) {
                sv.rng[id] = make_int2((int)r.x, (int)r.y);
                if (!reach_only) {
                    sv.rid[id] = (int)r.z;
                    sv.par[id] = from;
                    sv.acc[id] = shared || from == p0 || from == p1 ? (int)0x80000000 : 0;
                }
            }
        }
        q.head = (q.head + k) & (kRing - 1);
        q.n -= k;
    }
};

// Items in flight per lane: edge quads (independent cascade: one Philox block decides 4
// edges), or edges (linear threshold: a block per edge, keyed by its target).
template <bool kLT>
struct Items {
    static constexpr int N = kItems;
    int at[N];         // quad, or edge
    int src[N];        // local id of the row's vertex
    uint32_t ok[N];    // quad: its edges inside the row; edge: 1 inside
    uint32_t code[kLT ? 1 : N];
    uint32_t hi[kLT ? N : 1], lo[kLT ? N : 1], tgt[kLT ? N : 1];
};

template <bool kLT>
__device__ __forceinline__ void load_items(const TreeCall &c, Items<kLT> &it)
{
#pragma unroll
    for (int u = 0; u < Items<kLT>::N; ++u) {
        if constexpr (kLT) {
            it.hi[u] = it.lo[u] = it.tgt[u] = 0;
            if (it.ok[u]) {
                const uint32_t *thr = reinterpret_cast<const uint32_t *>(glob(c.thr4));
                const uint32_t *tl = reinterpret_cast<const uint32_t *>(glob(c.tl));
                const size_t e = (size_t)it.at[u];
                it.hi[u] = thr[e];
                it.tgt[u] = tl[((e >> 2) << 3) + (e & 3)];
                it.lo[u] = tl[((e >> 2) << 3) + (e & 3) + 4];
            }
        } else {
            it.code[u] = 0;
            if (it.ok[u]) it.code[u] = glob(c.code)[it.at[u]];
        }
    }
}

// The items' live edges (independent cascade: those that pass the test of the codes).
template <bool kLT>
__device__ __forceinline__ void decide(const TreeCall &c, const Items<kLT> &it, uint32_t j,
                                       uint32_t (&m)[Items<kLT>::N])
{
    // opaque here, so that the ten round keys are added up where they are used instead of
    // being kept in twenty scalar registers (the loop around this would spill them)
    uint32_t k0 = c.key_lo, k1 = c.key_hi;
    asm volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
    for (int u = 0; u < Items<kLT>::N; ++u) {
        if constexpr (kLT) {
            const uint32_t r = vertex_choice(it.tgt[u], j, k0, k1);
            m[u] = (r >= it.lo[u] && r < it.hi[u]) ? 1u : 0u;
        } else {
            uint32_t w0, w1, w2, w3;
            philox4x32_10((uint32_t)it.at[u], j, k0, k1, w0, w1, w2, w3);
            const uint32_t t = it.code[u];
            m[u] = ((coin_code(w0 >> 8) <= (int)(t & 0xFFu) ? 1u : 0u) |
                    (coin_code(w1 >> 8) <= (int)((t >> 8) & 0xFFu) ? 2u : 0u) |
                    (coin_code(w2 >> 8) <= (int)((t >> 16) & 0xFFu) ? 4u : 0u) |
                    (coin_code(w3 >> 8) <= (int)(t >> 24) ? 8u : 0u)) & it.ok[u];
        }
    }
}

// Append the items' edges to the queue in order; full batches are consumed.
template <bool kLT, class Sink>
__device__ __forceinline__ void enqueue(Sink &sink, WaveQueue &q, const int (&at)[Items<kLT>::N],
                                        const int (&src)[Items<kLT>::N],
                                        uint32_t (&m)[Items<kLT>::N], uint32_t j,
                                        uint32_t &live)
{
    constexpr int N = Items<kLT>::N;
    // positions by item number, then lane: at most 256 of each number, two counts in a word
    int pos[N];
    int found = 0;
#pragma unroll
    for (int u = 0; u < N; u += 2) {
        const int c0 = __builtin_popcount(m[u]), c1 = __builtin_popcount(m[u + 1]);
        const int incl = wave_scan(c0 | (c1 << 16));
        const int tot = __builtin_amdgcn_readlane(incl, 63);
        pos[u] = found + (incl & 0xFFFF) - c0;
        found += tot & 0xFFFF;
        pos[u + 1] = found + (incl >> 16) - c1;
        found += tot >> 16;
    }
    int done = 0;
    while (done < found) {
        const int room = min(found - done, kRing - q.n);
        const int off = q.head + q.n - done;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            while (m[u] && pos[u] < done + room) {
                const int i = __builtin_ctz(m[u]);
                m[u] &= m[u] - 1;
                const int slot = (off + pos[u]) & (kRing - 1);
                q.qe[slot] = (uint32_t)(kLT ? at[u] : (at[u] << 2) + i);
                q.qs[slot] = src[u];
                ++pos[u];
            }
        }
        wave_sync();
        q.n += room;
        done += room;
        while (q.n >= 64) sink.consume(q, 64, j, live);
        wave_sync();
    }
}

// Expand one level, the frontier [lo, hi): the seeds (source: the merged seed, local id 0) or
// local ids. Waves take chunks of the frontier, at most 64 vertices, from the level's counter
// and need no barrier until the level ends: claims and local ids are LDS atomics. A row of
// more than kHeavy items is left to a second pass in which all waves share it. Returns the
// number of vertices claimed.
template <int B, bool kLT, class Sink>
__device__ __forceinline__ int expand_level(const TreeCall &c, const int2 *rng, TreeHead<B> &sh,
                                            Sink &sink, bool from_seeds, int lo, int hi, int lset,
                                            uint32_t j, uint32_t &scanned, uint32_t &live)
{
    constexpr int W = B / 64;
    constexpr int N = Items<kLT>::N;
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    WaveQueue q{sh.qe[wid], sh.qs[wid], 0, 0};
    uint8_t *mark = sh.mark[wid];
    // several waves: at least four chunks each, so that they end together
    const int csz = W == 1 ? 64 : max(8, min(64, (hi - lo) / (4 * W)));
    int nh = -1;            // heavy rows of the level, once the first pass is over
    int h = 0, part = wid;  // this wave's next part of them: parts go round the waves
    // the rows at hand, one a lane: [e0, e1), items before them; the first lane's source
    int e0 = 0, e1 = 0, pre = 0, items = 0, total = 0, src0 = 0;
    // The next rows; false when the pass has none left.
    auto next_rows = [&]() {
        e0 = e1 = items = 0;
        if (nh < 0) {
            int k = 0;
            if (lane == 0) k = atomicAdd(&sh.chunk[lset], csz);
            src0 = lo + __builtin_amdgcn_readfirstlane(k);
            if (src0 >= hi) return false;
            k = src0 + lane;
            if (lane < csz && k < hi) {
                if (from_seeds) {
                    const int v = glob(c.seeds)[k];
                    e0 = glob(c.row_ptr)[v];
                    e1 = glob(c.row_ptr)[v + 1];
                } else {
                    const int2 r = rng[k];
                    e0 = r.x;
                    e1 = r.y;
                }
            }
            scanned += (uint32_t)(e1 - e0);
            items = kLT ? e1 - e0 : quads_of(e0, e1);
            if (W > 1 && items > kHeavy) {
                const int x = atomicAdd(&sh.nheavy[lset], 1);
                if (x < kHeavyCap) {
                    sh.heavy[0][x] = e0;
                    sh.heavy[1][x] = e1;
                    sh.heavy[2][x] = k;
                    items = 0;
                }
            }
        } else {
            // lane 0 holds the wave's next part of a heavy row
            int f0 = 0, f1 = 0, parts = 0;
            for (; h < nh; ++h) {
                f0 = __builtin_amdgcn_readfirstlane(sh.heavy[0][h]);
                f1 = __builtin_amdgcn_readfirstlane(sh.heavy[1][h]);
                parts = ((kLT ? f1 - f0 : quads_of(f0, f1)) + kPart - 1) / kPart;
                if (part < parts) break;
                part -= parts;
            }
            if (h >= nh) return false;
            const int first = kLT ? f0 + part * kPart : (f0 & ~3) + part * (4 * kPart);
            src0 = __builtin_amdgcn_readfirstlane(sh.heavy[2][h]);
            e0 = max(f0, first);
            e1 = part + 1 == parts ? f1 : first + (kLT ? kPart : 4 * kPart);
            items = lane == 0 ? (kLT ? e1 - e0 : quads_of(e0, e1)) : 0;
            part += W;
        }
        const int incl = wave_scan(items);
        pre = incl - items;
        total = __builtin_amdgcn_readlane(incl, 63);
        return true;
    };
    // Items sub + 64 u + lane of the rows: each row marks the item it begins at, and a running
    // maximum over the items gives each its row.
    auto place = [&](int sub, Items<kLT> &it) {
#pragma unroll
        for (int u = 0; u < N; ++u) mark[64 * u + lane] = 0;
        wave_sync();
        const bool begins = items > 0 && pre >= sub && pre < sub + 64 * N;
        if (begins) mark[pre - sub] = (uint8_t)lane;
        int run = 63 - __builtin_clzll(__ballot(items > 0 && pre <= sub) | 1ull);
        wave_sync();
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int i = sub + 64 * u + lane;
            const int l = max(run, wave_scan_max((int)mark[64 * u + lane]));
            run = __builtin_amdgcn_readlane(l, 63);
            const int f0 = __shfl(e0, l, 64), f1 = __shfl(e1, l, 64);
            const int d = i - __shfl(pre, l, 64);
            it.src[u] = from_seeds ? 0 : src0 + l;
            if constexpr (kLT) {
                it.at[u] = f0 + d;
                it.ok[u] = i < total ? 1u : 0u;
            } else {
                const int quad = (f0 >> 2) + d;
                const int eb = quad << 2;
                uint32_t ok = 0xFu;
                if (eb < f0) ok &= 0xFu << ((f0 - eb) & 3);
                if (eb + 4 > f1) ok &= 0xFu >> ((eb + 4 - f1) & 3);
                it.at[u] = quad;
                it.ok[u] = i < total ? ok : 0u;
            }
        }
        wave_sync();
    };
    for (;;) {
        while (!sink.full() && next_rows()) {
            Items<kLT> it;
            if (total > 0) {
                place(0, it);
                load_items<kLT>(c, it);
            }
            for (int sub = 0; sub < total; sub += 64 * N) {
                uint32_t m[N];
                int ats[N], srcs[N];
                decide<kLT>(c, it, j, m);
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    ats[u] = it.at[u];
                    srcs[u] = it.src[u];
                }
                // the next round's loads go out before this round's edges are followed
                if (sub + 64 * N < total) {
                    place(sub + 64 * N, it);
                    load_items<kLT>(c, it);
                }
                enqueue<kLT>(sink, q, ats, srcs, m, j, live);
            }
        }
        if (q.n > 0) {
            sink.consume(q, q.n, j, live);
            wave_sync();
        }
        __syncthreads();
        if (W == 1 || nh >= 0) break;
        nh = __builtin_amdgcn_readfirstlane(min(sh.nheavy[lset], kHeavyCap));
        if (nh == 0) break;
        sink.shared = true;
    }
    // the counters of the level before last: every wave is past reading them, and none
    // touches them again before the next level's barrier
    const int grown = sh.grown[lset];
    if (threadIdx.x == 0) {
        const int old = lset == 0 ? 2 : lset - 1;
        sh.chunk[old] = sh.grown[old] = sh.nheavy[old] = 0;
    }
    return grown;
}

// A subtree size into D: by reach id in single calls (folded into D by vertex once per
// launch, so that no add waits for a vertex id), by vertex in many-instance launches.
template <bool kMulti>
__device__ __forceinline__ void add_size(const TreeCall &c, int rid, int size)
{
    atomicAdd(&glob(c.D)[kMulti ? glob(c.rid_vtx)[rid] : rid], (unsigned long long)size);
}

// kMulti: every sample of the launch's list names its instance.
template <bool kMulti, bool kLT, int B>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(kTreeWaves, kTreeWaves)))
void tree_kernel(TreeArgs a)
{
    extern __shared__ __align__(16) unsigned char dyn[];
    TreeHead<B> &sh = *reinterpret_cast<TreeHead<B> *>(dyn);
    uint32_t *bm = reinterpret_cast<uint32_t *>(dyn + head_bytes<B>());
    const int tid = threadIdx.x, lane = lane_id();
    const size_t slot = blockIdx.x;
    TreeSlot sv;
    sv.rng = a.ws.rng + slot * (size_t)a.ws.lcap;
    sv.dom = reinterpret_cast<int32_t *>(sv.rng);
    sv.lid = sv.dom + a.ws.lcap;
    sv.rid = a.ws.rid + slot * (size_t)a.ws.lcap;
    sv.par = a.ws.par + slot * (size_t)a.ws.lcap;
    sv.acc = a.ws.acc + slot * (size_t)a.ws.lcap;
    sv.lvl = a.ws.lvl + slot * (size_t)(a.ws.lcap + 1);
    sv.extra = a.ws.extra + slot * (size_t)a.ws.xcap;
    sv.planes = a.ws.planes + slot * (size_t)(kTreePlanes * a.ws.words);
    const uint32_t *list = a.sample_list, *insts = a.sample_inst;
    uint32_t count = list ? *a.sample_count : a.theta;
    if (kMulti && a.alt_count && *a.alt_count <= a.alt_most) {
        list = a.alt_list;
        insts = a.alt_inst;
        count = *a.alt_count;
    }
    // samples whose dominator and size steps run in LDS: 6 bytes a vertex over everything
    // behind the scalars
    unsigned char *const over = dyn + free_offset<B>();
    const int lds_v = min(65535, (int)((a.lds_bytes - free_offset<B>()) / 6));

    uint32_t counted = 0;  // samples in the slot's planes
    int largest = 0;       // sample
    unsigned long long t_samples = 0, t_reached = 0, t_scanned = 0, t_live = 0;
    uint32_t cur = 0xFFFFFFFFu;
    TreeCall c{a.row_ptr, a.edge, a.code, a.thr4, a.tl, a.seeds, a.rid_vtx, a.nseeds, a.nclaim,
               a.nreach, a.key_lo, a.key_hi, a.D, a.stats, 0};

    auto flush_stats = [&]() {
        const unsigned long long sc = t_scanned, lv = t_live;
        unsigned long long s1 = sc, s2 = lv;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            s1 += __shfl_xor(s1, o, 64);
            s2 += __shfl_xor(s2, o, 64);
        }
        if (lane == 0) {
            if (s1) atomicAdd(&glob(c.stats)[2], s1);
            if (s2) atomicAdd(&glob(c.stats)[3], s2);
        }
        if (tid == 0 && t_samples) {
            atomicAdd(&glob(c.stats)[0], t_samples);
            atomicAdd(&glob(c.stats)[1], t_reached);
        }
        t_samples = t_reached = t_scanned = t_live = 0;
    };

    for (;;) {
        if (tid == 0) {
            sh.idx = atomicAdd(a.next, 1u);
            sh.nextra = 0;
            for (int i = 0; i < 3; ++i) sh.chunk[i] = sh.grown[i] = sh.nheavy[i] = 0;
        }
        __syncthreads();
        const uint32_t idx = sh.idx;
        if (idx >= count) break;
        const uint32_t j = list ? list[idx] : idx;
        if (kMulti) {
            const uint32_t i = __builtin_amdgcn_readfirstlane(insts[idx]);
            if (i != cur) {
                if (cur != 0xFFFFFFFFu) flush_stats();
                cur = i;
                const InstanceDesc &I = a.inst[i];
                const unsigned long long key =
                    (((unsigned long long)I.seed_hi << 32) | I.seed_lo) + a.round;
                c = TreeCall{scalar(I.row_ptr), scalar(I.tedge), scalar(I.code), scalar(I.thr4),
                             scalar(I.tl), scalar(I.seeds), scalar(I.rid_vtx),
                             scalar(I.nseeds), scalar(I.nclaim), scalar(I.nreach), scalar((uint32_t)key),
                             scalar((uint32_t)(key >> 32)), scalar(I.D), scalar(I.stats),
                             scalar(I.rec ? 0 : 1)};
            }
        }
        const int cwords = kLT ? 0 : (c.nclaim + 31) >> 5;
        for (int w = tid; w < cwords; w += B) bm[w] = 0u;
        if (tid == 0) {
            sv.lvl[0] = 0;
            sv.lvl[1] = 1;
        }
        __syncthreads();

        uint32_t p_scanned = 0, p_live = 0;
        int L = 0, lo = 0, hi = c.nseeds, base = 1, lset = 0;
        do {
            if (tid == 0 && L > 0) sv.lvl[L + 1] = hi;
            GroupSink<kLT> sink{c, sv, a.ws.xcap, a.reach_only != 0, bm, &sh.nextra, base,
                                &sh.grown[lset], false};
            const int grown = expand_level<B, kLT>(c, sv.rng, sh, sink, L == 0, lo, hi, lset, j,
                                                   p_scanned, p_live);
            lset = lset == 2 ? 0 : lset + 1;
            lo = base;
            base += grown;
            hi = base;
            ++L;
        } while (lo < hi);
        __syncthreads();
        const int nV = base;
        const int nX = kLT ? 0 : sh.nextra;
        if (nX > a.ws.xcap) {
            // more extra edges than the slot holds: the sample is re-run in large scratch
            if (tid == 0) {
                if (a.spill_ok) {
                    const uint32_t pos = atomicAdd(a.ovf_count, 1u);
                    a.ovf_list[pos] = j;
                    if (kMulti) a.ovf_inst[pos] = cur;
                    atomicAdd(&glob(c.stats)[4], 1ull);
                } else {
                    atomicOr(a.error, 1u);
                }
            }
            __syncthreads();
            continue;
        }
        t_scanned += p_scanned;
        t_live += p_live;
        if (tid == 0) {
            t_samples += 1;
            t_reached += (unsigned long long)(nV - 1);
            largest = max(largest, nV - 1);
        }
        if (a.reach_only || nV == 1) {
            __syncthreads();
            continue;
        }

        // Each reached vertex's own 1. A sample that reaches at least one vertex per two
        // bitmap words adds its bitmap to the slot's counters (the pass reads every word);
        // a smaller one leaves its ones to the D atomics below.
        const bool sliced = !kMulti && a.count_reach && (int64_t)nV * 64 >= c.nreach;
        if (sliced) {
            if (counted == kTreePlaneMax) {
                planes_drain<B>(sv.planes, a.ws.words, c.D);
                counted = 0;
                __syncthreads();
            }
            ++counted;
            // reach ids below nclaim are in the bitmap already
            const int64_t full = (int64_t)c.nclaim >> 5;
            if (!kLT) plane_add<B>(sv.planes, a.ws.words, 0, bm, (int)full);
            // the others one LDS bitmap at a time; the word that nclaim falls into is shared,
            // so its claimed bits are carried over
            const int64_t from = kLT ? 0 : full;
            for (int64_t r0 = from; r0 < a.ws.words; r0 += a.bm_words) {
                const int nw = (int)min<int64_t>(a.bm_words, a.ws.words - r0);
                const uint32_t carry = (!kLT && r0 == full && (c.nclaim & 31)) ? bm[full] : 0u;
                __syncthreads();
                for (int w = tid; w < nw; w += B) bm[w] = w == 0 ? carry : 0u;
                __syncthreads();
                for (int i = 1 + tid; i < nV; i += 4 * B) {
                    int r[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) r[u] = sv.rid[min(i + u * B, nV - 1)];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int64_t w = (r[u] >> 5) - r0;
                        if ((kLT || r[u] >= c.nclaim) && w >= 0 && w < nw)
                            atomicOr(&bm[w], 1u << (r[u] & 31));
                    }
                }
                __syncthreads();
                plane_add<B>(sv.planes, a.ws.words, r0, bm, nw);
            }
            __syncthreads();
        }

        // Extra edges: the target's reach id -> its local id. Mark the targets in the bitmap,
        // let each marked vertex leave its local id, then look them up.
        if (nX > 0) {
            for (int w = tid; w < cwords; w += B) bm[w] = 0u;
            __syncthreads();
            for (int x = tid; x < nX; x += B) {
                const uint32_t r = (uint32_t)sv.extra[x].y;
                atomicOr(&bm[r >> 5], 1u << (r & 31));
            }
            __syncthreads();
            for (int i = 1 + tid; i < nV; i += 4 * B) {
                uint32_t r[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) r[u] = (uint32_t)sv.rid[min(i + u * B, nV - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (r[u] < (uint32_t)c.nclaim && ((bm[r[u] >> 5] >> (r[u] & 31)) & 1u))
                        sv.lid[r[u]] = min(i + u * B, nV - 1);
            }
            __syncthreads();
            for (int x = tid; x < nX; x += B) {
                int4 e = sv.extra[x];
                e.y = sv.lid[e.y];
                e.z = sv.par[e.y];
                sv.extra[x] = e;
            }
            __syncthreads();
        }

        const int deep = sv.lvl[2];
        if (nV <= lds_v) {
            int *sz = reinterpret_cast<int *>(over);
            uint16_t *dom = reinterpret_cast<uint16_t *>(over + 4 * (size_t)nV);
            for (int i = tid; i < nV; i += B) {
                dom[i] = i ? (uint16_t)sv.par[i] : (uint16_t)0;
                sz[i] = 1;
            }
            __syncthreads();
            while (nX > 0) {
                if (tid == 0) sh.changed = 0;
                __syncthreads();
                for (int x = tid; x < nX; x += B) {
                    const int4 e = sv.extra[x];
                    const int tv = ld(&dom[e.y]);
                    if (tv == 0) continue;
                    const int m = tree_nca(dom, deep, tree_nca(dom, deep, tv, e.x), e.z);
                    if (m < tv) {
                        st(&dom[e.y], (uint16_t)m);
                        sh.changed = 1;
                    }
                }
                __syncthreads();
                const int ch = sh.changed;
                __syncthreads();
                if (!ch) break;
            }
            for (int l = L - 1; l > 1; --l) {
                const int b0 = sv.lvl[l], b1 = sv.lvl[l + 1];
                for (int i = b0 + tid; i < b1; i += B) {
                    const int t = dom[i];
                    if (t != 0) atomicAdd(&sz[t], sz[i]);
                }
                __syncthreads();
            }
            for (int i = 1 + tid; i < nV; i += 4 * B) {
                int add[4], r[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = i + u * B;
                    add[u] = k < nV ? sz[k] - (sliced ? 1 : 0) : 0;
                    r[u] = add[u] > 0 ? sv.rid[k] : 0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (add[u] > 0) add_size<kMulti>(c, r[u], add[u]);
            }
            __syncthreads();
        } else {
            // The tentative dominators take the place of the parents of extra edges' targets
            // while they are raised; then such a vertex gets its parent back, with the sign
            // bit set when its dominator differs, which is left in dom[].
            while (nX > 0) {
                if (tid == 0) sh.changed = 0;
                __syncthreads();
                for (int x = tid; x < nX; x += B) {
                    const int4 e = sv.extra[x];
                    const int tv = ld(&sv.par[e.y]);
                    if (tv == 0) continue;
                    const int m = tree_nca(sv.par, deep, tree_nca(sv.par, deep, tv, e.x), e.z);
                    if (m < tv) {
                        st(&sv.par[e.y], m);
                        sh.changed = 1;
                    }
                }
                __syncthreads();
                const int ch = sh.changed;
                __syncthreads();
                if (!ch) break;
            }
            if (nX > 0) {
                for (int x = tid; x < nX; x += B) {
                    const int4 e = sv.extra[x];
                    sv.extra[x].w = ld(&sv.par[e.y]);
                }
                __syncthreads();
                for (int x = tid; x < nX; x += B) {
                    const int4 e = sv.extra[x];
                    if (e.w != e.z) {
                        st(&sv.par[e.y], e.z | (int)0x80000000);
                        sv.dom[e.y] = e.w;
                    }
                }
                __syncthreads();
            }
            // Subtree sizes, deepest level first. A wave sums the runs of equal parents over 64
            // vertices. An unmarked run that lies inside them holds all children of its parent
            // and is the only writer of that sum; a marked or cut one is added with an atomic,
            // as is a vertex whose dominator is not its parent (that dominator is at least two
            // levels above, where no run of this level ends).
            constexpr int U = 4;  // vertices in flight per lane
            for (int l = L - 1; l > 1; --l) {
                const int b0 = sv.lvl[l], b1 = sv.lvl[l + 1];
                for (int j0 = b0 + U * (tid & ~63); j0 < b1; j0 += U * B) {
                    int pu[U], su[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = j0 + 64 * u + lane;
                        pu[u] = i < b1 ? sv.par[i] : 0;
                        su[u] = i < b1 ? ld(&sv.acc[i]) : 0;
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i0 = j0 + 64 * u;
                        if (i0 >= b1) break;
                        const int i = i0 + lane;
                        const bool in = i < b1;
                        const bool moved = pu[u] < 0, shared = su[u] < 0;
                        const int p = pu[u] & 0x7FFFFFFF;
                        const int s = in ? (su[u] & 0x7FFFFFFF) + 1 : 0;
                        const int incl = wave_scan(moved ? 0 : s);
                        const int pp = __shfl_up(p, 1, 64), pn = __shfl_down(p, 1, 64);
                        const bool head = in && (lane == 0 || pp != p);
                        const bool last = in && (i + 1 >= b1 || lane == 63 || pn != p);
                        const unsigned long long hm = __ballot(head);
                        const int h = 63 - __builtin_clzll((hm & (~0ull >> (63 - lane))) | 1ull);
                        const int upto = __shfl(incl, max(h - 1, 0), 64);
                        if (last) {
                            const int sum = incl - (h > 0 ? upto : 0);
                            const bool cut = shared || (h == 0 && i0 > b0) || (lane == 63 && i + 1 < b1);
                            if (sum > 0) {
                                if (cut)
                                    __hip_atomic_fetch_add(&sv.acc[p], sum, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                                else
                                    st(&sv.acc[p], ld(&sv.acc[p]) + sum);
                            }
                        }
                        if (moved) {
                            const int t = sv.dom[i];
                            if (t != 0)
                                __hip_atomic_fetch_add(&sv.acc[t], s, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                    }
                }
                __syncthreads();
            }
            for (int i = 1 + tid; i < nV; i += 4 * B) {
                int add[4], r[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = i + u * B;
                    add[u] = k < nV ? (ld(&sv.acc[k]) & 0x7FFFFFFF) + (sliced ? 0 : 1) : 0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) r[u] = add[u] > 0 ? sv.rid[i + u * B] : 0;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (add[u] > 0) add_size<kMulti>(c, r[u], add[u]);
            }
            __syncthreads();
        }
    }
    if (!kMulti || cur != 0xFFFFFFFFu) flush_stats();
    if (!kMulti && tid == 0) {
        if (a.count_reach) a.ws.used[slot] = counted;
        if (largest > 0) atomicMax(&a.stats[kStatLargest], (unsigned long long)largest);
    }
}

// The same for samples of at most kLeafV vertices: one wavefront per sample, sixteen samples
// per compute unit, everything but the row ranges and the extra edges in 10 KB of LDS, and no
// barrier. Reach ids are claimed in a hash table (independent cascade). What bounds such
// samples is latency: a level costs the row ranges, the codes and the records one after the
// other, so what counts is how many samples are in flight. A sample that outgrows the space
// is handed over to the workgroup kernel, with nothing accumulated.
constexpr int kLeafV = 576;      // local vertices, root included
constexpr int kLeafX = 512;      // extra edges
constexpr int kLeafHash = 1024;
constexpr int kLeafLevels = 120;
constexpr uint32_t kLeafRun = 16;  // samples taken at a time, at most

struct LeafShared {
    TreeHead<64> h;
    uint16_t lvl[kLeafLevels + 2];
    uint16_t par[kLeafV];        // BFS parents, then dominators
    uint16_t slot[kLeafV];       // hash slot of each local vertex
    int4 key[kLeafHash / 4];     // reach ids: by hash slot (-1: empty); linear threshold: by
                                 // local id
    union {
        uint16_t lid[kLeafHash]; // local id by hash slot
        int size[kLeafV];        // once the extra edges are resolved
    };
};
static_assert(sizeof(LeafShared) <= kTreeLds / 16, "sixteen samples per compute unit");

template <bool kLT>
struct LeafSink {
    const TreeCall &c;
    LeafShared &sm;
    int *key;
    int2 *rng;
    int4 *extra;
    bool reach_only;
    int tail = 1, nextra = 0;
    bool over = false;
    bool shared = false;

    __device__ __forceinline__ bool full() const { return over; }

    __device__ __forceinline__ void consume(WaveQueue &q, int k, uint32_t j, uint32_t &live)
    {
        const int lane = lane_id();
        if (tail + k > kLeafV) over = true;
        if (!over) {
            uint4 r;
            int from;
            const bool has = follow<kLT>(c, q, lane < k, j, r, from);
            live += has ? 1u : 0u;
            bool won = has;
            uint32_t h = 0;
            if (!kLT && has) {
                // at most kLeafV of the kLeafHash slots are ever taken
                h = (r.z * 2654435761u) >> 22;
                for (;;) {
                    const int old = atomicCAS(&key[h], -1, (int)r.z);
                    won = old == -1;
                    if (won || old == (int)r.z) break;
                    h = (h + 1) & (kLeafHash - 1);
                }
            }
            const unsigned long long below = (1ull << lane) - 1ull;
            const unsigned long long b = __ballot(won);
            if (won) {
                const int id = tail + __builtin_popcountll(b & below);
                rng[id] = make_int2((int)r.x, (int)r.y);
                sm.par[id] = (uint16_t)from;
                if (kLT) {
                    key[id] = (int)r.z;
                } else {
                    sm.slot[id] = (uint16_t)h;
                    sm.lid[h] = (uint16_t)id;
                }
            }
            tail += __builtin_popcountll(b);
            if (!kLT && !reach_only) {
                const bool x = has && !won && from != 0;
                const unsigned long long bx = __ballot(x);
                const int at = nextra + __builtin_popcountll(bx & below);
                if (x && at < kLeafX) extra[at] = make_int4(from, (int)h, 0, 0);
                nextra += __builtin_popcountll(bx);
                if (nextra > kLeafX) over = true;
            }
        }
        q.head = (q.head + k) & (kRing - 1);
        q.n -= k;
    }
};

// One sample; false when it must be handed over.
template <bool kLT>
__device__ __forceinline__ bool leaf_sample(const TreeCall &c, LeafShared &sm, int2 *rng,
                                            int4 *extra, bool reach_only, uint32_t j,
                                            uint32_t &scanned, uint32_t &live, int &reached)
{
    const int lane = lane_id();
    wave_sync();
    int *const key = reinterpret_cast<int *>(sm.key);
    if (!kLT) {
#pragma unroll
        for (int i = 0; i < kLeafHash / 256; ++i) sm.key[i * 64 + lane] = make_int4(-1, -1, -1, -1);
    }
    if (lane < 3) sm.h.chunk[lane] = sm.h.grown[lane] = sm.h.nheavy[lane] = 0;
    if (lane == 0) {
        sm.lvl[0] = 0;
        sm.lvl[1] = 1;
        sm.par[0] = 0;
    }
    wave_sync();
    LeafSink<kLT> sink{c, sm, key, rng, extra, reach_only};
    int L = 0, lo = 0, hi = c.nseeds, lset = 0;
    do {
        if (L >= kLeafLevels) return false;
        if (lane == 0 && L > 0) sm.lvl[L + 1] = (uint16_t)hi;
        const int base = sink.tail;
        expand_level<64, kLT>(c, rng, sm.h, sink, L == 0, lo, hi, lset, j, scanned, live);
        if (sink.over) return false;
        lset = lset == 2 ? 0 : lset + 1;
        lo = base;
        hi = sink.tail;
        ++L;
    } while (lo < hi);
    wave_sync();
    const int nV = sink.tail, nX = sink.nextra;
    reached = nV - 1;
    if (reach_only || nV == 1) return true;

    if (!kLT && nX > 0) {
        for (int x = lane; x < nX; x += 64) {
            int4 e = extra[x];
            e.y = sm.lid[e.y];
            e.z = sm.par[e.y];
            extra[x] = e;
        }
        wave_sync();
        const int deep = sm.lvl[2];
        for (;;) {
            bool changed = false;
            for (int x = lane; x < nX; x += 64) {
                const int4 e = extra[x];
                const int tv = ld(&sm.par[e.y]);
                if (tv == 0) continue;
                const int m = tree_nca(sm.par, deep, tree_nca(sm.par, deep, tv, e.x), e.z);
                if (m < tv) {
                    st(&sm.par[e.y], (uint16_t)m);
                    changed = true;
                }
            }
            wave_sync();
            if (!__any(changed)) break;
        }
    }
    int *size = sm.size;
    for (int i = lane; i < nV; i += 64) size[i] = 1;
    wave_sync();
    for (int l = L - 1; l > 1; --l) {
        const int b0 = sm.lvl[l], b1 = sm.lvl[l + 1];
        for (int i = b0 + lane; i < b1; i += 64) {
            const int t = sm.par[i];
            if (t != 0) atomicAdd(&size[t], size[i]);
        }
        wave_sync();
    }
    for (int i = 1 + lane; i < nV; i += 64) {
        const int rid = key[kLT ? i : sm.slot[i]];
        atomicAdd(&glob(c.D)[glob(c.rid_vtx)[rid]], (unsigned long long)size[i]);
    }
    return true;
}

template <bool kMulti, bool kLT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kTreeWaves, kTreeWaves)))
void leaf_kernel(LeafArgs a)
{
    __shared__ LeafShared sm;
    const int lane = lane_id();
    int2 *rng = a.rng + (size_t)blockIdx.x * kLeafV;
    int4 *extra = a.extra + (size_t)blockIdx.x * kLeafX;
    const uint32_t count = a.sample_list ? *a.sample_count : a.total;
    if (kMulti && count <= a.leave) return;
    uint32_t cur = 0xFFFFFFFFu, cur_lo = 0, cur_hi = 0;
    bool skip = false, done = false;
    TreeCall c{};
    uint32_t *ctrl = nullptr;
    unsigned long long t_samples = 0, t_reached = 0, t_scanned = 0, t_live = 0;
    auto flush_stats = [&]() {
        unsigned long long s1 = t_scanned, s2 = t_live;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            s1 += __shfl_xor(s1, o, 64);
            s2 += __shfl_xor(s2, o, 64);
        }
        if (lane == 0 && t_samples) {
            atomicAdd(&glob(c.stats)[0], t_samples);
            atomicAdd(&glob(c.stats)[1], t_reached);
            atomicAdd(&glob(c.stats)[2], s1);
            atomicAdd(&glob(c.stats)[3], s2);
            atomicAdd(&glob(c.stats)[5], t_samples);
        }
        t_samples = t_reached = t_scanned = t_live = 0;
    };
    auto hand_over = [&](uint32_t j) {
        if (lane == 0) {
            const bool low = kMulti && c.nreach <= a.low_reach;
            const uint32_t at = atomicAdd(low ? a.low_count : a.out_count, 1u);
            (low ? a.low_j : a.out_j)[at] = j;
            if (kMulti) (low ? a.low_inst : a.out_inst)[at] = cur;
        }
    };
    uint32_t seen = 0;
    for (;;) {
        // runs of consecutive samples that shrink as the launch drains
        uint32_t first = 0, last = 0;
        if (lane == 0) {
            const uint32_t left = seen < count ? count - seen : 0u;
            const uint32_t want = max(1u, min(kLeafRun, left / (4u * gridDim.x)));
            first = atomicAdd(a.next, want);
            last = min(first + want, count);
        }
        first = __builtin_amdgcn_readfirstlane(first);
        last = __builtin_amdgcn_readfirstlane(last);
        if (first >= last) break;
        seen = last;
        for (uint32_t idx = first; idx < last; ++idx) {
            uint32_t inst = 0, j = idx;
            if (a.sample_list) {
                j = __builtin_amdgcn_readfirstlane(a.sample_list[idx]);
                if (kMulti) inst = __builtin_amdgcn_readfirstlane(a.sample_inst[idx]);
            } else if (kMulti) {
                inst = cur;
                if (cur == 0xFFFFFFFFu || idx < cur_lo || idx >= cur_hi) {
                    int lo = 0, hi = a.ninst - 1;
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (a.inst[mid].sample_base <= idx) lo = mid;
                        else hi = mid - 1;
                    }
                    inst = __builtin_amdgcn_readfirstlane(lo);
                }
            }
            if (inst != cur) {
                if (cur != 0xFFFFFFFFu) flush_stats();
                cur = inst;
                const InstanceDesc &I = a.inst[inst];
                const unsigned long long key =
                    (((unsigned long long)I.seed_hi << 32) | I.seed_lo) + a.round;
                c = TreeCall{scalar(I.row_ptr), scalar(I.tedge), scalar(I.code), scalar(I.thr4),
                             scalar(I.tl), scalar(I.seeds), scalar(I.rid_vtx),
                             scalar(I.nseeds), scalar(I.nclaim), scalar(I.nreach),
                             scalar((uint32_t)key), scalar((uint32_t)(key >> 32)), scalar(I.D),
                             scalar(I.stats), scalar(I.rec ? 0 : 1)};
                if (kMulti) {
                    ctrl = scalar(I.ctrl);
                    cur_lo = scalar(I.sample_base);
                    cur_hi = cur_lo + scalar(I.theta);
                    // an instance that handed most samples of an earlier round over skips this
                    // kernel; the samples of one whose run has ended are dropped
                    skip = __builtin_amdgcn_readfirstlane(ld(&ctrl[kCtrlSkipWave])) != 0u;
                    done = __builtin_amdgcn_readfirstlane(ld(&ctrl[kCtrlDone])) != 0u;
                }
            }
            if (kMulti && !a.sample_list) j = idx - cur_lo;
            if (kMulti && done) continue;
            uint32_t scanned = 0, live = 0;
            int reached = 0;
            if (!(kMulti && skip) &&
                leaf_sample<kLT>(c, sm, rng, extra, a.reach_only != 0, j, scanned, live, reached)) {
                t_samples += 1;
                t_reached += (unsigned long long)reached;
                t_scanned += scanned;
                t_live += live;
            } else {
                hand_over(j);
                if (kMulti && !skip && lane == 0) atomicAdd(&ctrl[kCtrlWaveHanded], 1u);
            }
        }
    }
    if (cur != 0xFFFFFFFFu) flush_stats();
}

// D[v] += the sizes by reach id (Dr) and the bit-sliced reach counts of every slot that kept
// some (used), which go back to 0.
// A workgroup takes 16 bitmap words (512 reach ids) and shares the slots of its part (grid y)
// among 16 thread rows; each thread adds its slots' planes into a bit-sliced sum and the rows
// meet in LDS counters, so D is touched once per vertex and part.
constexpr int kDrainWords = 16;
constexpr int kDrainRows = 16;
constexpr int kDrainBits = 20;  // 63 samples in each of at most 4096 slots

__global__ __launch_bounds__(kDrainWords *kDrainRows) void drain_planes_kernel(
    uint32_t *planes, const uint32_t *used, int32_t slots, int64_t words, const int32_t *rid_vtx,
    int32_t nreach, const unsigned long long *Dr, unsigned long long *D)
{
    __shared__ uint32_t sum[kDrainWords * 32];
    const int wd = threadIdx.x % kDrainWords, row = threadIdx.x / kDrainWords;
    for (int i = threadIdx.x; i < kDrainWords * 32; i += kDrainWords * kDrainRows) sum[i] = 0u;
    __syncthreads();
    const int64_t w = (int64_t)blockIdx.x * kDrainWords + wd;
    uint32_t s[kDrainBits];
#pragma unroll
    for (int i = 0; i < kDrainBits; ++i) s[i] = 0u;
    if (w < words) {
        for (int32_t sl = blockIdx.y * kDrainRows + row; sl < slots; sl += gridDim.y * kDrainRows) {
            const uint32_t n = used[sl];
            if (!n) continue;
            uint32_t *at = planes + (size_t)sl * kTreePlanes * words + w;
            uint32_t p[kTreePlanes];
#pragma unroll
            for (int i = 0; i < kTreePlanes; ++i) p[i] = (n >> i) ? at[i * words] : 0u;
            uint32_t carry = 0;
#pragma unroll
            for (int i = 0; i < kDrainBits; ++i) {
                const uint32_t x = i < kTreePlanes ? p[i] : 0u;
                const uint32_t o = s[i];
                s[i] = o ^ x ^ carry;
                carry = (o & x) | (carry & (o ^ x));
            }
#pragma unroll
            for (int i = 0; i < kTreePlanes; ++i)
                if (p[i]) at[i * words] = 0u;
        }
    }
    for (int b = 0; b < 32; ++b) {
        uint32_t v = 0;
#pragma unroll
        for (int i = 0; i < kDrainBits; ++i) v |= ((s[i] >> b) & 1u) << i;
        if (v) atomicAdd(&sum[wd * 32 + b], v);
    }
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * kDrainWords * 32;
    for (int i = threadIdx.x; i < kDrainWords * 32 && r0 + i < nreach; i += kDrainWords * kDrainRows) {
        const unsigned long long v = sum[i] + (blockIdx.y == 0 && Dr ? Dr[r0 + i] : 0ull);
        if (v) atomicAdd(&D[rid_vtx[r0 + i]], v);
    }
}

// Per edge: the target's row range, its reach id and the edge's threshold; the threshold's
// code; the record without a threshold (target, its row range) of the other kernels; the working
// threshold; and, per quad, its targets and lower bounds. Null outputs are left out.
__global__ void edge_records_kernel(const uint32_t *col, const int32_t *row_ptr, const int32_t *rid,
                                    const uint32_t *thr, const uint32_t *lo, int64_t m,
                                    int64_t padded, uint4 *edge, uint8_t *code, uint4 *plain,
                                    uint32_t *work, uint32_t *tl)
{
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < padded;
         e += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t v = col[e], t = thr[e];
        work[e] = t;
        if (tl) {
            uint32_t *const at = tl + (e >> 2) * 8 + (e & 3);
            at[0] = v;
            at[4] = lo[e];
        }
        if (e >= m) continue;
        const uint32_t r0 = (uint32_t)row_ptr[v], r1 = (uint32_t)row_ptr[v + 1];
        if (edge) edge[e] = make_uint4(r0, r1, (uint32_t)rid[v], t);
        if (code) code[e] = (uint8_t)threshold_code(t);
        if (plain) plain[e] = make_uint4(v, r0, r1, 0u);
    }
}

// Every record's threshold as created.
__global__ void edge_restore_kernel(const uint32_t *thr, int64_t m, uint4 *edge)
{
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * blockDim.x)
        edge[e].w = thr[e];
}

// The workgroup size to take where several keep all the waves at work that the registers allow.
// A small workgroup waits less for itself at level ends and runs more samples at once; a large
// one ends the launch's largest sample sooner, and that is what a launch of few or of very
// different samples waits for. What is known before the call is the samples per slot of 512
// threads, the size of the graph, and the seeds' out-edges, which bound nothing but go with the
// samples' sizes (few: most samples end at once, some reach thousands). Kernel times in ms, by
// threads; 2^n: R-MAT graphs of so many vertices, their seeds drawn at random unless said.
//   * Linear threshold, reachability too, where 128 was taken once: 10,000 samples from 20 seeds
//     of 2^20 25.7 with 128, 8.8 with 512; from 100 seeds of a 262k-vertex Chung-Lu graph 7.9 and
//     6.0. Few samples a slot and few seeds: 2,000 from 20 seeds of 2^20 9.1 with 512, 7.2 with
//     1024; on graphs as large also 10,000 from one seed, 1.82 and 1.52.
//   * Reachability: 64, but 256 from few seeds of a graph with large samples: 10,000 from 20 seeds
//     of 2^17 1.17 and 0.82, but from its 10 largest vertices 4.5 and 5.2; and 512 from few seeds
//     of the next larger graphs: 10,000 from one of 2^19 1.15 with 256, 0.83 with 512, but 20,000
//     from 20 2.7 and 3.4.
//   * Dominators: 512. Few samples a slot from few seeds of a large graph: 1024; 2,000 from 20
//     seeds of 2^19 1.65 and 1.37, from 100 of 2^18 1.26 and 1.25, from 100 of 2^17 1.04 and 1.33.
//     Many samples a slot: 256; 10,000 from 100 seeds of 2^17 3.6 and 3.0, of 2^19 7.2 and 5.9, of
//     a 40k-vertex trivalency graph 0.49 and 0.38, but from 20 seeds of 2^17 0.94 and 1.16, and
//     from its 10 largest vertices 9.3 and 9.5. From 64 a slot on also from fewer seeds: 50,000
//     from 20 of 2^17 2.4 and 1.9, but from one 0.92 and 1.24. Graphs of a few thousand vertices
//     have no large samples: from 20 seeds of 1,000 vertices 10,000 take 0.87 and 0.59, 50,000
//     3.8, 2.1 and, with 128, 1.4.
int32_t preferred_block(const TreeFit &f)
{
    const int64_t slots = 2 * (int64_t)std::max(1, f.num_cus), e = f.seed_edges;
    if (f.lt) {
        const bool few = f.nreach > (1 << 16) && e <= 4096 && f.theta <= 4 * slots;
        const bool one = f.nreach > (1 << 18) && e <= 512 && f.theta <= 64 * slots;
        return e >= 0 && (few || one) ? 1024 : 512;
    }
    if (f.reach_only) {
        if (e < 0 || e > 512 || f.nreach <= (1 << 15)) return 64;
        return f.nreach > 3 * (1 << 16) && f.theta <= 32 * slots ? 512 : 256;
    }
    if (e < 0 || e > 16384) return 512;
    if (f.nreach > (1 << 16) && e <= (f.nreach > (1 << 17) ? 1024 : 512) && f.theta <= 4 * slots)
        return 1024;
    const bool tiny = f.nreach <= 4096;
    if (f.theta >= 64 * slots && e >= 32) return tiny ? 128 : 256;
    return f.theta >= 16 * slots && e >= (tiny ? 64 : 512) ? 256 : 512;
}

// The shape with workgroups of B threads, if it has more threads at work on the samples than the
// best so far.
template <int B>
void shape_for(int64_t bits, const TreeFit &f, TreeShape &best, int64_t &best_threads)
{
    // whole shares of LDS are multiples of 16 bytes
    const size_t need = head_bytes<B>() + ((size_t)((bits + 31) / 32) * 4 + 15) / 16 * 16;
    if (need > kTreeLds) return;
    const int wgs = (int)std::min<size_t>(256 * kTreeWaves / B, kTreeLds / need);
    int64_t at_work = std::min<int64_t>(f.theta, (int64_t)wgs * f.num_cus);
    if (f.most > 0) at_work = std::min(at_work, f.most);
    const int64_t threads = at_work * B;
    if (threads <= best_threads) return;
    best_threads = threads;
    best.block = B;
    best.per_cu = wgs;
    // the whole share: what the bitmap leaves goes to the dominator steps
    best.lds = (uint32_t)(kTreeLds / wgs / 16 * 16);
    best.bm_words = (int32_t)((best.lds - head_bytes<B>()) / 4);
}

template <bool kMulti, bool kLT>
hipError_t launch_shape(const TreeArgs &a, const TreeShape &s, hipStream_t stream)
{
    const dim3 grid(a.ws.slots);
    void (*k)(TreeArgs) = nullptr;
    if (s.block == 512) k = tree_kernel<kMulti, kLT, 512>;
    else if (s.block == 1024) k = tree_kernel<kMulti, kLT, 1024>;
    if constexpr (!kMulti) {  // many-instance launches prefer 512, and take 1024 where that is more
        if (s.block == 64) k = tree_kernel<kMulti, kLT, 64>;
        else if (s.block == 128) k = tree_kernel<kMulti, kLT, 128>;
        else if (s.block == 256) k = tree_kernel<kMulti, kLT, 256>;
    }
    if (!k) return hipErrorInvalidValue;
    const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)s.lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k, grid, dim3(s.block), s.lds, stream, a);
    return hipGetLastError();
}

}  // namespace

int leaf_slots(int num_cus) { return 16 * std::max(1, num_cus); }

size_t leaf_slot_bytes() { return kLeafV * sizeof(int2) + kLeafX * sizeof(int4); }

hipError_t launch_leaf(const LeafArgs &args, unsigned char *scratch, int slots, bool multi, bool lt,
                       hipStream_t stream)
{
    if (slots <= 0 || !scratch) return hipErrorInvalidValue;
    LeafArgs a = args;
    a.extra = reinterpret_cast<int4 *>(scratch);
    a.rng = reinterpret_cast<int2 *>(scratch + (size_t)slots * kLeafX * sizeof(int4));
    if (!multi && !lt) return hipErrorInvalidValue;  // single calls: linear threshold alone
    void (*k)(LeafArgs) = !multi ? leaf_kernel<false, true>
                          : lt   ? leaf_kernel<true, true>
                                 : leaf_kernel<true, false>;
    hipLaunchKernelGGL(k, dim3(slots), dim3(64), 0, stream, a);
    return hipGetLastError();
}

// A greedy run's later rounds know the first one's samples. Where none is large, small workgroups
// do them all, and the threads at work count for less. Eight rounds, kernel times in ms, trivalency
// graphs: 2,000 samples of 222 vertices 1.48 with 64 threads, 2.04 with 512; of 758 (1,000 at the
// most) 2.31 with 256, 2.72 with 512, 500 of those 1.16 with 256, 1.63 with 1024, and 1,000 1.57 with
// 128, 1.79 with 256; 10,000 of 28 2.85 with 64, 2.45 with 128, 3.10 with 512; of 12 2.15 with 256,
// 2.38 with 512, but of one 1.79 and 1.46. Twelve rounds, whole calls: 1,000 samples of 19 1.25 with
// 64, 1.82 with 512, but 2,000 of 25 1.97 and 1.66.
int32_t block_after(const TreeFit &f, double mean, uint64_t largest)
{
    const int64_t slots = 2 * (int64_t)std::max(1, f.num_cus);
    if (largest > 4096) return 0;
    if (largest > 512)
        return mean < 48.0 ? 0 : mean < 1024.0 && f.theta > slots && f.theta <= 2 * slots ? 128 : 256;
    if (f.theta >= 16 * slots && mean < 64.0) return mean >= 16.0 ? 128 : mean >= 6.0 ? 256 : 0;
    return mean >= (f.theta > 2 * slots ? 32.0 : 16.0) ? 64 : 0;
}

bool tree_shape(const TreeFit &f, TreeShape &out)
{
    int64_t threads = 0;
    out = TreeShape{};
    // linear threshold: the bitmap only counts, a part of the reach ids at a time
    const int64_t cap = (int64_t)(kTreeLds - head_bytes<1024>()) * 8;
    const int64_t bits = f.lt ? std::min((f.nreach + 3) / 4, cap) : f.nclaim;
    auto consider = [&](int32_t b) {
        if (b == 64) shape_for<64>(bits, f, out, threads);
        else if (b == 128) shape_for<128>(bits, f, out, threads);
        else if (b == 256) shape_for<256>(bits, f, out, threads);
        else if (b == 512) shape_for<512>(bits, f, out, threads);
        else shape_for<1024>(bits, f, out, threads);
    };
    // A size that block_after gave. And 512 where that many slots take the samples at once, and 1024
    // threads would have to take them in turns on as many compute units: 500 samples from the 10
    // largest of 40,111 vertices (weighted cascade, 9,770 vertices each) 0.47 ms with 512, 0.58
    // with 1024; not for samples of few seeds (50: 0.12 and 0.09, trivalency), nor on larger graphs
    // (500 from 100 seeds of 2^18 R-MAT vertices 0.98 and 0.73).
    const int64_t slots = 2 * (int64_t)std::max(1, f.num_cus);
    const bool at_once = !f.lt && !f.reach_only && f.theta <= slots && f.theta > slots / 2 &&
                         f.seed_edges >= 2048 && f.nreach <= (1 << 16);
    if (!f.block && (f.prefer || at_once)) {
        consider(f.prefer ? f.prefer : 512);
        if (out.per_cu * out.block >= kTreeLeast) return true;
    }
    for (int32_t b : {preferred_block(f), 64, 128, 256, 512, 1024})
        if (!f.block || b == f.block) consider(b);
    if (f.block == 0 && out.per_cu * out.block < kTreeLeast) out = TreeShape{};
    return out.block > 0;
}

hipError_t launch_tree(const TreeArgs &args, const TreeShape &s, bool lt, hipStream_t stream)
{
    if (args.ws.slots <= 0 || s.block == 0) return hipErrorInvalidValue;
    TreeArgs a = args;
    a.lds_bytes = s.lds;
    a.bm_words = s.bm_words;
    // many-instance launches: independent cascade (the forest kernel and the kernel of
    // decrease.hip take linear threshold)
    if (a.inst) return lt ? hipErrorInvalidValue : launch_shape<true, false>(a, s, stream);
    return lt ? launch_shape<false, true>(a, s, stream) : launch_shape<false, false>(a, s, stream);
}

hipError_t launch_drain_planes(const TreeWs &ws, int32_t slots, const int32_t *rid_vtx,
                               int32_t nreach, const unsigned long long *Dr, unsigned long long *D,
                               hipStream_t stream)
{
    if (slots <= 0 || nreach <= 0) return hipSuccess;
    const int64_t bx = (ws.words + kDrainWords - 1) / kDrainWords;
    const int by = (int)std::max<int64_t>(1, std::min<int64_t>(8, 512 / bx));
    hipLaunchKernelGGL(drain_planes_kernel, dim3((uint32_t)bx, by), dim3(kDrainWords * kDrainRows), 0,
                       stream, ws.planes, ws.used, slots, ws.words, rid_vtx, nreach, Dr, D);
    return hipGetLastError();
}

hipError_t launch_edge_records(const uint32_t *col, const int32_t *row_ptr, const int32_t *rid,
                               const uint32_t *thr, const uint32_t *lo, int64_t m, int64_t padded,
                               uint4 *edge, uint8_t *code, uint4 *plain, uint32_t *work, uint32_t *tl,
                               hipStream_t stream)
{
    const int grid = (int)std::min<int64_t>(8192, (padded + 255) / 256);
    hipLaunchKernelGGL(edge_records_kernel, dim3(grid), dim3(256), 0, stream, col, row_ptr, rid, thr,
                       lo, m, padded, edge, code, plain, work, tl);
    return hipGetLastError();
}

hipError_t launch_edge_restore(const uint32_t *thr, int64_t m, uint4 *edge, hipStream_t stream)
{
    if (m <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>(8192, (m + 255) / 256);
    hipLaunchKernelGGL(edge_restore_kernel, dim3(grid), dim3(256), 0, stream, thr, m, edge);
    return hipGetLastError();
}

}  // namespace imin
