// forest.hip -- Algorithm 2 of arXiv 2302.13529 under the linear-threshold model (Section V-E),
// from the side of the chosen in-edges.
//
// In a sample every vertex keeps at most one in-edge, so the sampled graph is a forest hanging
// from the seeds plus trees that hang from vertices without a choice or from cycles. A reached
// vertex's only path comes through its chosen in-edge: that edge is its dominator-tree edge,
// its subtree is its dominator subtree, and there is nothing to claim and no extra edge.
//
// Expanding the reached vertices' out-edges draws one choice per scanned edge, 15 to 18 times
// as many as there are reached vertices on R-MAT graphs, of which a large sample reaches more
// than half anyway. So for graphs whose vertices fit LDS (reach ids below 65,533) a workgroup
// draws each vertex's choice once and follows it up:
//   1. choices. Lanes take consecutive reach ids. The chosen in-edge is the first whose bound
//      exceeds the draw; the guess draw * degree / 2^24, which is right where the weights of a
//      vertex are equal, is tried first, then a binary search. The in-edges are 4-byte words
//      (16 bits of the bound, 16 of the source); a draw that ties in those 16 bits is decided
//      by the exact bound. The whole of a 131k-vertex graph's words fits an XCD's L2;
//   2. reach, by doubling in place: a vertex's entry is an ancestor of it and becomes that
//      one's entry. Seeds and the absence of a parent are their own ancestors. A sweep that
//      brings no vertex to a seed is the last: the shallowest vertex still on its way points at
//      one that has arrived, so it would arrive;
//   3. sizes, by doubling over the reached vertices: in round r a vertex holds its 2^r-th
//      ancestor and the number of its descendants nearer than 2^r, and adds the latter to the
//      former's in LDS. No order of the vertices is needed, and the number of rounds is the
//      logarithm of the depth (R-MAT samples are 60 levels deep). Sums stay below 2^16, so two
//      share a word and never carry;
//   4. counts. The reached set goes into the slot's bit-sliced counters (single calls), sizes
//      above 1 into D, consecutive lanes to consecutive counters.
// LDS holds one array of 16-bit entries, ancestors and sums in turn, beside the bitmaps.
// The sizes pass keeps its ancestors and sizes in registers: kept in memory they were read and
// written every round, beyond the L2 with all slots at work, and a launch took 7.2 ms for 4.4. In
// the forms of 32 words a thread they do not all fit beside what else lives: the compiler spills 11
// registers in single calls (17 with 1,024 threads) and 8 in many-instance launches of 1,024.
//
// What bounds it is the random reads of the choices (L2) and of the doubling rounds (LDS).
// Measured with 5,000 samples of a 131k-vertex R-MAT graph that reach 35,300 vertices each:
// 20.4 ms with the workgroup kernel's expansion, 9.4 with depths found by sweeps over the
// chosen edges and a list sorted by depth, 5.1 so. 32 graphs of 1,000 to 50,000 vertices, ten
// rounds of GreedyReplace: 152 to 75 ms.
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

// The thread's first index, hidden from the optimiser: known, the addresses of every pass over
// the entries are computed once for all samples and kept in registers, more than there are.
__device__ __forceinline__ int own(int tid)
{
    asm volatile("" : "+v"(tid));
    return tid;
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

// Parent codes: a reach id, nreach for a seed (its own parent), nreach + 1 for none.
constexpr uint32_t kNoRid = 0xFFFD;  // in-edge words: the source has no reach id

struct ForestHead {
    uint32_t idx;
    int changed;
    int reached;
    int pad;
};

struct ForestCall {
    const uint4 *node;
    const uint32_t *in16;
    const uint32_t *bound;
    const int32_t *src;
    const int32_t *rid_of;
    const uint32_t *inelig;
    const int32_t *seeds;
    int32_t nseeds, nreach, nsrc;
    uint32_t key_lo, key_hi;
    unsigned long long *D;
    unsigned long long *stats;
};

// In-edge e's bound exceeds the draw r.
__device__ __forceinline__ bool below(const ForestCall &c, uint32_t word, uint32_t e, uint32_t r)
{
    const uint32_t hi = word >> 16, r16 = r >> 8;
    return r16 < hi || (r16 == hi && r < glob(c.bound)[e]);
}

// Parent code of the node (vertex v, in-edges [first, first + deg)) in sample j.
__device__ __forceinline__ uint32_t choose(const ForestCall &c, const uint32_t *srcbits, uint4 node,
                                           uint32_t r)
{
    const uint32_t first = node.y, deg = node.z;
    uint32_t k = min((uint32_t)(((uint64_t)r * deg) >> 24), deg - 1);
    uint32_t word = glob(c.in16)[first + k];
    const uint32_t prev = k ? glob(c.in16)[first + k - 1] : 0u;
    if (!below(c, word, first + k, r)) {
        uint32_t lo = k + 1, hi = deg;  // the first below() in [lo, hi), or hi
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (below(c, glob(c.in16)[first + mid], first + mid, r)) hi = mid;
            else lo = mid + 1;
        }
        if (lo == deg) return (uint32_t)c.nreach + 1;
        k = lo;
        word = glob(c.in16)[first + k];
    } else if (k && below(c, prev, first + k - 1, r)) {
        uint32_t lo = 0, hi = k - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (below(c, glob(c.in16)[first + mid], first + mid, r)) hi = mid;
            else lo = mid + 1;
        }
        k = lo;
        word = glob(c.in16)[first + k];
    }
    const uint32_t s = word & 0xFFFFu;
    if (s != kNoRid) return s;
    const int32_t at = glob(c.src)[first + k];
    return (srcbits[at >> 5] >> (at & 31)) & 1u ? (uint32_t)c.nreach : (uint32_t)c.nreach + 1;
}

// Words of two vertices each, for nreach vertices and the two codes: whole turns of B threads, by
// fours.
__host__ __device__ constexpr int forest_entries(int B, int nreach)
{
    return (nreach / 2 + 4 * B) / (4 * B) * (4 * B);
}

// KW words a thread at the most.
template <bool kMulti, int B, int KW>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(4, 4)))
void forest_kernel(ForestArgs a)
{
    extern __shared__ __align__(16) unsigned char dyn[];
    ForestHead &sh = *reinterpret_cast<ForestHead *>(dyn);
    uint32_t *const mask = reinterpret_cast<uint32_t *>(dyn + sizeof(ForestHead));  // seeds, blocked
    const int tid = threadIdx.x, lane = lane_id();
    const size_t slot = blockIdx.x;
    uint32_t *const parent = a.ws.parent + slot * (size_t)a.ws.entries;
    uint32_t *const my_planes = a.ws.planes + slot * (size_t)(kTreePlanes * a.ws.words);
    const uint32_t count = a.sample_list ? *a.sample_count : a.theta;
    uint32_t counted = 0, cur = 0xFFFFFFFFu;
    unsigned long long t_samples = 0, t_reached = 0, t_scanned = 0;
    uint32_t seed_scan = 0;  // out-edges of the seeds, a share per thread
    ForestCall c{};
    int words = 0, swords = 0;

    auto flush_stats = [&]() {
        unsigned long long s = t_scanned;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0 && s) atomicAdd(&glob(c.stats)[2], s);
        if (tid == 0 && t_samples) {
            atomicAdd(&glob(c.stats)[0], t_samples);
            atomicAdd(&glob(c.stats)[1], t_reached);
            atomicAdd(&glob(c.stats)[3], t_reached);  // a reached vertex's one live in-edge
        }
        t_samples = t_reached = t_scanned = 0;
    };

    for (;;) {
        if (tid == 0) {
            sh.idx = atomicAdd(a.next, 1u);
            sh.reached = 0;
        }
        __syncthreads();
        const uint32_t idx = sh.idx;
        if (idx >= count) break;
        const uint32_t j = a.sample_list ? a.sample_list[idx] : idx;
        const uint32_t inst = kMulti ? (uint32_t)__builtin_amdgcn_readfirstlane(a.sample_inst[idx]) : 0u;
        if (inst != cur) {
            if (cur != 0xFFFFFFFFu) flush_stats();
            cur = inst;
            const InstanceDesc &I = a.inst[inst];
            const unsigned long long key =
                (((unsigned long long)I.seed_hi << 32) | I.seed_lo) + a.round;
            c = ForestCall{I.fnode, I.fin16, I.fbound, I.fsrc, I.rid_of, I.inelig, I.seeds,
                           I.nseeds, I.nreach, I.nsrc, (uint32_t)key, (uint32_t)(key >> 32),
                           kMulti ? I.D : a.Dr, I.stats};
            words = (c.nreach + 31) >> 5;
            swords = (c.nsrc + 31) >> 5;
            // the masked reach ids, and the seeds among the sources without one
            uint32_t *const bits = mask + 2 * words;
            for (int w = tid; w < words; w += B) mask[w] = 0u;
            for (int w = tid; w < swords; w += B) bits[w] = 0u;
            __syncthreads();
            for (int u = tid; u < c.nreach; u += B) {
                const uint32_t v = glob(c.node)[u].x;
                if ((glob(c.inelig)[v >> 5] >> (v & 31)) & 1u) atomicOr(&mask[u >> 5], 1u << (u & 31));
            }
            seed_scan = 0;
            for (int k = tid; k < c.nseeds; k += B) {
                const int v = glob(c.seeds)[k], r = glob(c.rid_of)[v];
                seed_scan += (uint32_t)(glob(I.row_ptr)[v + 1] - glob(I.row_ptr)[v]);
                if (r < 0) atomicOr(&bits[(-1 - r) >> 5], 1u << ((-1 - r) & 31));
            }
            __syncthreads();
        }
        uint32_t *const reach = mask + words;
        uint32_t *const srcbits = reach + words;
        uint32_t *const arr = srcbits + swords;
        uint16_t *const half = reinterpret_cast<uint16_t *>(arr);

        const uint32_t root = (uint32_t)c.nreach, none = root + 1;
        const int nw = forest_entries(B, c.nreach);

        // 1. every vertex's choice; the entries behind the vertices are their own
        for (int u0 = own(tid); u0 < c.nreach; u0 += 4 * B) {
            uint4 nd[4];
            uint32_t p[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) nd[i] = glob(c.node)[min(u0 + i * B, c.nreach - 1)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int u = min(u0 + i * B, c.nreach - 1);
                const uint32_t r = vertex_choice(nd[i].x, j, c.key_lo, c.key_hi);
                p[i] = (mask[u >> 5] >> (u & 31)) & 1u ? none : choose(c, srcbits, nd[i], r);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (u0 + i * B < c.nreach) half[u0 + i * B] = (uint16_t)p[i];
        }
        for (int u = c.nreach + own(tid); u < 2 * nw; u += B)
            half[u] = (uint16_t)(u == (int)root ? root : none);
        __syncthreads();
        // the seeds with a reach id are their own roots
        for (int k = tid; k < c.nseeds; k += B) {
            const int r = glob(c.rid_of)[glob(c.seeds)[k]];
            if (r >= 0) half[r] = (uint16_t)root;
        }
        __syncthreads();
        for (int w = own(tid); w < nw; w += B) parent[w] = arr[w];

        // 2. reach
        for (;;) {
            __syncthreads();
            if (tid == 0) sh.changed = 0;
            __syncthreads();
            bool now = false;
#pragma unroll 4
            for (int w = own(tid); w < nw; w += B) {
                const uint32_t e = ld(&arr[w]);
                uint32_t x = e & 0xFFFFu, y = e >> 16;
                if (x < root) x = ld(&half[x]);
                if (y < root) y = ld(&half[y]);
                const uint32_t f = x | (y << 16);
                if (f != e) {
                    st(&arr[w], f);
                    now = now || (x == root && (e & 0xFFFFu) != root) || (y == root && (e >> 16) != root);
                }
            }
            if (now) sh.changed = 1;
            __syncthreads();
            if (!sh.changed) break;
        }
        // the vertices at a seed, seeds (masked) aside
        int mine = 0;
        for (int u = own(tid); u < 2 * nw; u += B) {
            const bool in = u < c.nreach && half[u] == root && !((mask[u >> 5] >> (u & 31)) & 1u);
            if (in) t_scanned += glob(c.node)[u].w;
            mine += in ? 1 : 0;
            const unsigned long long b = __ballot(in);
            if ((lane & 31) == 0 && (u >> 5) < words) reach[u >> 5] = (uint32_t)(b >> lane);
        }
        const int all = wave_scan(mine);
        if (lane == 63 && all) atomicAdd(&sh.reached, all);
        __syncthreads();
        const int nR = sh.reached;
        if (tid == 0) {
            t_samples += 1;
            t_reached += (unsigned long long)nR;
        }
        t_scanned += seed_scan;
        if (a.reach_only || nR == 0) {
            __syncthreads();
            continue;
        }

        // 3. sizes: anc and size hold two vertices a word, the unreached as root and 0. They stay
        // in registers; in memory they would be read and written in every round, more than the
        // L2 of all slots holds. Words beyond the graph's are skipped four at a time.
        uint32_t anc[KW], size[KW];
        uint32_t *const own_words = arr + own(tid);
#pragma unroll
        for (int i = 0; i < KW; ++i) {
            const int w = own(tid) + i * B;
            const uint32_t in = (w >> 4) < words ? reach[w >> 4] >> ((w & 15) * 2) & 3u : 0u;
            const uint32_t p = i * B < nw ? parent[w] : 0u;
            anc[i] = (in & 1u ? p & 0xFFFFu : root) | ((in & 2u ? p >> 16 : root) << 16);
            size[i] = (in & 1u) | ((in >> 1) << 16);
            if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
        for (;;) {
            for (int w = own(tid); w < nw; w += B) arr[w] = 0u;
            if (tid == 0) sh.changed = 0;
            __syncthreads();
#pragma unroll
            for (int g = 0; g < KW; g += 4) {
                if (g * B < nw)
#pragma unroll
                for (int i = g; i < g + 4; ++i) {
                    asm volatile("" : "+v"(anc[i]), "+v"(size[i]));
                    const uint32_t x = anc[i] & 0xFFFFu, y = anc[i] >> 16;
                    if (x != root) atomicAdd(&arr[x >> 1], (size[i] & 0xFFFFu) << ((x & 1) * 16));
                    if (y != root) atomicAdd(&arr[y >> 1], (size[i] >> 16) << ((y & 1) * 16));
                }
            }
            __syncthreads();
#pragma unroll
            for (int g = 0; g < KW; g += 4) {
                if (g * B < nw)
#pragma unroll
                for (int i = g; i < g + 4; ++i) {
                    asm volatile("" : "+v"(anc[i]), "+v"(size[i]));
                    const uint32_t add = own_words[i * B], z = size[i];
                    // what fell on a seed's entry is nobody's
                    const uint32_t in = (z & 0xFFFFu ? 0xFFFFu : 0u) | (z >> 16 ? 0xFFFF0000u : 0u);
                    size[i] = z + (add & in);
                    own_words[i * B] = anc[i];
                }
            }
            __syncthreads();
            bool more = false;
#pragma unroll
            for (int g = 0; g < KW; g += 4) {
                if (g * B < nw)
#pragma unroll
                for (int i = g; i < g + 4; ++i) {
                    asm volatile("" : "+v"(anc[i]), "+v"(size[i]));
                    uint32_t x = anc[i] & 0xFFFFu, y = anc[i] >> 16;
                    if (x != root) x = half[x];
                    if (y != root) y = half[y];
                    anc[i] = x | (y << 16);
                    more = more || x != root || y != root;
                }
            }
            if (more) sh.changed = 1;
            __syncthreads();
            const int ch = sh.changed;
            __syncthreads();
            if (!ch) break;
        }

        // 4. counts
        const bool sliced = !kMulti && a.ws.words > 0 && (int64_t)nR * 64 >= c.nreach;
        if (sliced) {
            if (counted == kTreePlaneMax) {
                planes_drain<B>(my_planes, a.ws.words, c.D);
                counted = 0;
                __syncthreads();
            }
            ++counted;
            plane_add<B>(my_planes, a.ws.words, 0, reach, words);
        }
        const uint32_t off = sliced ? 1u : 0u;
#pragma unroll
        for (int g = 0; g < KW; g += 4) {
            if (g * B < nw)
#pragma unroll
            for (int i = g; i < g + 4; ++i) {
                asm volatile("" : "+v"(anc[i]), "+v"(size[i]));
                const uint32_t u = 2u * (uint32_t)(own(tid) + i * B);
                const uint32_t x = size[i] & 0xFFFFu, y = size[i] >> 16;
                if (x > off)
                    atomicAdd(&glob(c.D)[kMulti ? glob(c.node)[u].x : u], (unsigned long long)(x - off));
                if (y > off)
                    atomicAdd(&glob(c.D)[kMulti ? glob(c.node)[u + 1].x : u + 1],
                              (unsigned long long)(y - off));
            }
        }
        __syncthreads();
    }
    if (cur != 0xFFFFFFFFu) flush_stats();
    if (!kMulti && tid == 0 && a.ws.words > 0) a.ws.used[slot] = counted;
}

// The in-edge words, one in-edge a thread; its source is the row it lies in. In a host loop this
// took half of a graph's creation (131k vertices: 21.7 ms; 9.6 without the index).
__global__ void forest_index_kernel(const int32_t *in_ptr, const int32_t *in_edge, const uint32_t *col,
                                    const int32_t *row_ptr, int32_t n, int32_t m, const int32_t *rid,
                                    const uint32_t *bound, const uint4 *node, uint32_t *in16,
                                    uint32_t *exact, int32_t *src)
{
    for (int64_t k = blockIdx.x * 256ll + threadIdx.x; k < m; k += (int64_t)gridDim.x * 256) {
        const int32_t e = in_edge[k];
        const uint32_t v = col[e], b = bound[e];
        int32_t lo = 0, hi = n - 1;  // the last row that starts at or before e
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo + 1) / 2;
            if (row_ptr[mid] <= e) lo = mid;
            else hi = mid - 1;
        }
        const int32_t r = rid[lo];
        const uint32_t at = node[rid[v]].y + (uint32_t)(k - in_ptr[v]);
        in16[at] = ((b ? b - 1 : 0u) >> 8 << 16) | (r >= 0 ? (uint32_t)r : kNoRid);
        exact[at] = b;
        src[at] = r >= 0 ? lo : -1 - r;
    }
}

template <int B, int KW>
bool class_for(int64_t nreach, int64_t nsrc, ForestShape &out)
{
    const int entries = forest_entries(B, (int)nreach);
    if (entries > B * KW) return false;
    const size_t need = sizeof(ForestHead) +
                        (size_t)(2 * ((nreach + 31) / 32) + (nsrc + 31) / 32 + entries) * 4;
    const size_t lds = (need + 255) / 256 * 256;
    if (lds > kTreeLds) return false;
    out.block = B;
    out.words = KW;
    out.entries = entries;
    out.lds = (uint32_t)lds;
    out.per_cu = (int32_t)std::min<size_t>(256 * kTreeWaves / B, kTreeLds / lds);
    return true;
}

}  // namespace

// The smallest workgroup with which a compute unit runs all the waves its registers hold: more
// samples at once hide one's barriers. Larger arrays leave room for fewer, larger workgroups.
bool forest_shape(int64_t nreach, int64_t nsrc, ForestShape &out)
{
    out = ForestShape{};
    if (nreach <= 0 || nreach >= (int64_t)kNoRid) return false;
    const int full = 256 * kTreeWaves;
    if (class_for<256, 16>(nreach, nsrc, out) && out.per_cu * out.block >= full) return true;
    if (class_for<256, 32>(nreach, nsrc, out) && out.per_cu * out.block >= full) return true;
    if (class_for<512, 32>(nreach, nsrc, out) && out.per_cu * out.block >= full) return true;
    return class_for<1024, 32>(nreach, nsrc, out);
}

hipError_t launch_forest_index(const int32_t *in_ptr, const int32_t *in_edge, const uint32_t *col,
                               const int32_t *row_ptr, int32_t n, int32_t m, const int32_t *rid,
                               const uint32_t *bound, const uint4 *node, uint32_t *in16,
                               uint32_t *exact, int32_t *src, hipStream_t stream)
{
    if (m <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>(4096, ((int64_t)m + 255) / 256);
    hipLaunchKernelGGL(forest_index_kernel, dim3(grid), dim3(256), 0, stream, in_ptr, in_edge, col,
                       row_ptr, n, m, rid, bound, node, in16, exact, src);
    return hipGetLastError();
}

hipError_t launch_forest(const ForestArgs &a, const ForestShape &s, int slots, bool multi,
                         hipStream_t stream)
{
    if (slots <= 0 || s.block == 0) return hipErrorInvalidValue;
    void (*k)(ForestArgs) = nullptr;
    if (s.block == 256 && s.words == 16)
        k = multi ? forest_kernel<true, 256, 16> : forest_kernel<false, 256, 16>;
    else if (s.block == 256)
        k = multi ? forest_kernel<true, 256, 32> : forest_kernel<false, 256, 32>;
    else if (s.block == 512)
        k = multi ? forest_kernel<true, 512, 32> : forest_kernel<false, 512, 32>;
    else
        k = multi ? forest_kernel<true, 1024, 32> : forest_kernel<false, 1024, 32>;
    const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)s.lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k, dim3(slots), dim3(s.block), s.lds, stream, a);
    return hipGetLastError();
}

}  // namespace imin
