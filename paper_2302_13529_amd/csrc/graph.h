// graph.h -- the host-side graph handle of libimin and the helpers its C entry points share
// (api.cpp: single and batched calls; server.cpp: the query server).
#pragma once

#include "imin.h"
#include "imin_internal.h"

#include <algorithm>
#include <vector>

namespace imin {
namespace host {
struct MultiScratch;

// A call's share of the graph's pinned block.
struct CallPin {
    imin::InstanceDesc *inst = nullptr;  // sent
    int32_t *seeds = nullptr, *undo = nullptr, *mask = nullptr;
    uint32_t *inelig = nullptr, *cand = nullptr;
    unsigned long long *stats = nullptr, *D = nullptr;  // written by kernels
    uint32_t *ctrl = nullptr;
    int32_t *x = nullptr, *B = nullptr;
};
}  // namespace host
}  // namespace imin

struct imin_graph {
    int device = 0;
    int32_t n = 0;
    int32_t m = 0;
    int num_cus = 1;
    std::vector<int32_t> row_ptr;  // host copies: out-neighbours of the seeds (GR)
    std::vector<int32_t> col;
    unsigned char *block = nullptr;  // one allocation: every array below but the growing ones
                                  // (d_sj, d_ovf, d_B and the kernels' scratch)
    int32_t *d_row_ptr = nullptr;
    uint4 *d_col4 = nullptr;      // edge targets, 4 per quad, padded to a whole quad
    uint4 *d_edge = nullptr;      // independent cascade: one record per edge slot of d_col4,
                                  // (target, target's row start, row end, 0)
    uint4 *d_thr4 = nullptr;      // working live thresholds, same layout: 0 on every edge into
                                  // a vertex of `masked`
    uint4 *d_thr_orig = nullptr;  // the thresholds ceil(p * 2^24) as created
    int model = 0;                // IMIN_IC or IMIN_LT
    uint4 *d_lo4 = nullptr;       // linear-threshold model: interval lower bounds
    uint4 *d_tl = nullptr;        // linear-threshold model: per quad, its targets and then its
                                  // lower bounds (32 bytes, one line)
    int32_t nclaim = 0, nreach = 0;  // reach ids: first the vertices of two or more in-edges,
                                  // then those of one, each ascending
    int32_t *d_rid_vtx = nullptr; // nreach: vertex of each reach id
    bool tree = false;            // the LDS-claim kernel serves this graph
    imin::TreeShape shape;        // its launch shape in the current call
    uint4 *d_tedge = nullptr;     // its edge records (their thresholds masked as d_thr4) and
    uint32_t *d_code = nullptr;   // threshold codes
    // linear threshold, few enough reachable vertices: forest.hip's arrays (InstanceDesc)
    bool forest = false;
    imin::ForestShape fshape;
    int32_t nsrc = 0;
    uint4 *d_fnode = nullptr;
    uint32_t *d_fin16 = nullptr, *d_fbound = nullptr;
    int32_t *d_fsrc = nullptr, *d_rid_of = nullptr;
    int32_t *d_in_ptr = nullptr;  // in-edges of v: d_in_edge[d_in_ptr[v] .. d_in_ptr[v+1])
    int32_t *d_in_edge = nullptr; // edge ids, grouped by target
    hipStream_t stream = nullptr;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    int32_t words = 0;                       // 32-bit words of a vertex bitmap
    uint32_t *d_inelig = nullptr;            // seeds and blocked vertices
    uint32_t *d_cand = nullptr;              // GR candidate set CB
    int32_t *d_seeds = nullptr;              // distinct seeds (capacity n)
    unsigned long long *d_D = nullptr;       // n, then nreach by reach id
    unsigned long long *d_stats = nullptr;   // kStats: samples, reached, scanned, live,
                                             // spilled, wave-kernel samples
    uint32_t *d_ctrl = nullptr;              // kCtrlWords: next main, next spill, spill count,
                                             // error (in batched calls: the instance's words)
    uint32_t *d_sctrl = nullptr;             // 3: wave-kernel work counter, samples it left,
                                             // the next kernel's work counter
    unsigned char *pin = nullptr;            // pinned: what a call sends and what comes back
    size_t pin_cap = 0;
    imin::host::CallPin at;                  // the current call's share of it
    bool in_flight = false;                  // a call's end was not waited for
    int clock_khz = 0;                       // of the device's wall clock
    uint32_t *d_sj = nullptr;                // samples the wave kernel left to the large one
    uint32_t sj_cap = 0;
    imin::InstanceDesc *d_inst = nullptr;    // this graph as the one instance of a wave launch
    imin::InstanceDesc h_inst{};
    int small_mode = -1;                     // wave kernel: -1 automatic, 0 off, 1 on
    bool small_auto_off = false;             // automatic mode: this call's first round found
                                             // most samples too large
    bool auto_pending = false;               // wave kernel on: this call's first round not yet judged
    int probe = 0;                           // automatic mode, per call: 1 = time the next
                                             // round (wave kernel on), 2 = the next round is a
                                             // timed trial without it, 3 = compare; 0 = none
    size_t probe_kev[2] = {0, 0};            // kev index of the timed rounds (with, without)
    imin_launch small_launch{};              // 0 fields: defaults
    uint32_t *d_ovf = nullptr;
    uint32_t ovf_cap = 0;
    unsigned long long *d_part_d = nullptr;
    int32_t *d_part_i = nullptr;
    int32_t parts = 4096;
    int32_t *d_B = nullptr;
    int32_t B_cap = 0;
    int32_t *d_x = nullptr;
    imin::Workspace main_ws, big_ws;
    imin::TreeWs main_tw, big_tw;
    imin::TreeWs reach_tw;             // main_tw's space as slots of row ranges and level starts
    unsigned char *leaf = nullptr;     // the wave-per-sample form's scratch
    imin::ForestWs fws;
    std::vector<int32_t> masked;       // vertices whose in-edges have threshold 0 in d_thr4
    std::vector<int32_t> mask_prev;    // the previous call's list
    bool mask_known = true;            // false while a call runs, and after one that failed
    int32_t *d_list = nullptr;         // n: device copy of `masked`
    std::vector<hipEvent_t> kev;  // pairs around each decrease launch of the current call
    size_t kev_used = 0;
    imin::host::MultiScratch *batch_ms = nullptr;  // scratch of the batches this graph leads
                                                   // (first instance), kept for the next one
    // the records that masks also go to (the LDS-claim kernel's, independent cascade)
    uint4 *mask_rec() const { return model == IMIN_IC ? d_tedge : nullptr; }
    int32_t force_slots = 0;
    int64_t force_xcap = 0;
    int32_t force_block = 0;           // imin_set_workgroup
    int64_t seed_edges = -1;           // out-edges of the current call's seeds
    int32_t prefer = 0;                // TreeFit::prefer, for the current call's later rounds
    bool wave_first = false;           // automatic mode, LDS-claim kernel: many_small's choice
};

namespace imin {
namespace host {

constexpr int kClock = 7;  // behind the stats: a round's start, the rounds' time (clock ticks),
                           // kStatLargest
constexpr int kCallStats = kStatLargest + 1;
static_assert(kStatLargest == kClock + 2, "behind the clock");
constexpr int kStats = 7;  // samples, reached, scanned, live, spilled, wave-level kernel
                           // samples, packed-kernel samples
// The per-launch work counter is 32-bit and every workgroup takes one index past the end.
constexpr uint32_t kMaxTheta = 1u << 31;

inline bool ok(hipError_t e) { return e == hipSuccess; }

// The LDS-claim kernel, and before it the forest kernel, run this graph's single calls.
inline bool tree_on(const imin_graph *g)
{
    return g->tree && (g->force_block >= 0 || g->model == IMIN_LT);
}
// The shape of its launches over theta samples.
inline TreeFit tree_fit(const imin_graph *g, int64_t theta, bool reach_only)
{
    TreeFit f;
    f.nclaim = g->nclaim;
    f.nreach = g->nreach;
    f.lt = g->model == IMIN_LT;
    f.reach_only = reach_only;
    f.theta = theta;
    f.num_cus = g->num_cus;
    f.seed_edges = g->seed_edges;
    f.block = std::max(g->force_block, 0);
    f.prefer = g->prefer;
    return f;
}
inline int64_t out_edges(const imin_graph *g, const int32_t *S, size_t nS)
{
    int64_t sum = 0;
    for (size_t i = 0; i < nS; ++i) sum += g->row_ptr[(size_t)S[i] + 1] - g->row_ptr[(size_t)S[i]];
    return sum;
}
// Calls of the LDS-claim kernel with so many samples that the wave kernel takes the small ones
// first. 5,120 of those run at once in it, and in the other as many as there are slots; but it
// costs 0.25 ms at the least, and where most samples are large, a few of them on each wave before
// it gives up (many out-edges of the seeds make that likely). In ms without and with it:
//   * claims that leave one slot a compute unit: from 64 samples a slot on. 50,000 samples of a
//     1M-vertex Chung-Lu graph from one seed 4.1 and 3.3, from 20 13.6 and 10.7, from 100 (all
//     large) 35.9 and 36.9; 10,000 (39 a slot) from one 1.28 and 1.42;
//   * more slots: from 131,072 samples on. 200,000 of a 1M-vertex R-MAT graph from one seed 7.2
//     and 5.7, from 20 23.0 and 20.5; 50,000 of a 131k-vertex Chung-Lu graph 0.91 and 1.17. On
//     graphs of a few thousand vertices, whose smaller workgroups run 2,048 at once, and for
//     reachability (up to 4,096) only from seeds of hardly any out-edges: 200,000 samples of a
//     1,000-vertex graph from one seed 3.2 and 2.2, reachability on 2^17 R-MAT vertices 2.9 and 2.2.
inline bool many_small(const imin_graph *g, int64_t theta, int64_t slots, bool reach_only)
{
    const int64_t e = g->seed_edges;
    if (g->model != IMIN_IC || e < 0 || e > 4096) return false;
    if (slots <= g->num_cus) return theta >= 64 * slots;
    return theta >= 512 * (int64_t)g->num_cus && (e <= 64 || (!reach_only && g->nreach > 4096));
}
inline bool forest_on(const imin_graph *g) { return g->forest && g->force_block <= 0; }

template <class T>
void dfree(T *&p)
{
    if (p) (void)hipFree(p);
    p = nullptr;
}

// Extra edges a slot holds: a quarter of the vertices, reachable or not, and never more than
// there are edges. A sample with more runs again in one of the two large slots. 2,000 samples of
// a 1M-vertex R-MAT graph under trivalency, 60,800 vertices each: 48.6 ms, where a quarter of the
// vertices that have an in-edge sent them to the large slots and took 3,642.
inline int64_t extra_cap(int64_t n, int64_t m)
{
    return std::min(std::max<int64_t>(4096, (n + 1) / 4), m + 1);
}

void free_ws(Workspace &ws);
// Scratch of `slots` workgroup-kernel slots with maps of n entries (kept when the shape is
// unchanged); cleared on `stream`.
int alloc_ws(Workspace &ws, int64_t n, int32_t slots, int64_t lcap, int64_t xcap,
             hipStream_t stream);
// Validated seed set: distinct seeds ascending, and the seed bitmap.
int seed_setup(imin_graph *g, const int32_t *S, int32_t nS, std::vector<int32_t> &seeds,
               std::vector<uint32_t> &inelig);
// The arrays of `slots` tree-kernel slots carved from base (null: only counted); returns the
// bytes they take.
size_t carve_tree(TreeWs &ws, unsigned char *base, int32_t slots, int64_t lcap, int64_t xcap,
                  int64_t nclaim, int64_t words);
int small_grid(int num_cus, const imin_launch &l);
void small_shape(SmallArgs &s, const imin_launch &l);
bool launch_ok(const imin_launch *l);

// Where a workgroup-kernel launch reads its call state and accumulates: the graph's own
// buffers for single calls, a query's for the server.
struct LargeTarget {
    const uint4 *thr4;
    const int32_t *seeds;
    int32_t nseeds;
    unsigned long long *D;
    unsigned long long *stats;
    uint32_t *ctrl;      // 4 words: next main, next spill, spill count, error
    uint32_t *ovf;       // capacity >= theta
    Workspace *main_ws;  // slots > 0
    Workspace *big_ws;   // slots == 0 when no sample can overflow main_ws
    const TreeWs *main_tw;  // graphs of the LDS-claim kernel: these instead
    const TreeWs *big_tw;
    unsigned long long *Dr; // and its counters by reach id, zero when the launch starts
};
// The workgroup kernel over samples 0..theta-1, or over the device list `list` of *count
// samples, then the large-scratch launch for the samples that overflowed.
int launch_large_on(imin_graph *g, const LargeTarget &t, uint32_t theta, uint64_t key,
                    const uint32_t *list, const uint32_t *count, bool reach_only);

// Device scratch of rounds over many instances at once (batched calls, the server): the
// wave kernel's hand-over list, the workgroup kernel's slots (maps sized for the largest
// instance) and its own overflow list, and the control words of one round.
constexpr int kMultiCtrl = 10;

struct MultiScratch {
    int64_t n = 0, m = 0;      // largest instance it serves
    uint32_t cap = 0;          // samples of the largest round
    Workspace main_ws, big_ws;
    bool tree = false;         // the LDS-claim kernel takes the hand-overs instead, in these
    TreeShape shape;
    TreeWs main_tw, big_tw;
    unsigned char *leaf = nullptr;  // the wave-per-sample form's scratch
    bool forest = false;            // linear threshold: the forest kernel takes the hand-overs,
    bool split = false;             // the smaller graphs' in launches of their own
    ForestShape fshape, low_shape;
    ForestWs fws, low_ws;
    uint32_t *ctrl = nullptr;  // kMultiCtrl: wave next, wave hand-overs, wave error, main
                               // next, big next, overflow count, workgroup error, packed
                               // hand-overs, packed next, instances done this call
    uint32_t *pi = nullptr, *pj = nullptr;  // packed kernel's hand-over list: instance, sample
    uint32_t *si = nullptr, *sj = nullptr;  // wave kernel's hand-over list: instance, sample
    uint32_t *oi = nullptr, *oj = nullptr;  // overflow list: instance, sample
    int32_t inst_cap = 0;                   // instances of the largest round
    unsigned long long *part_d = nullptr;   // inst_cap * kArgParts partial argmax results
    int32_t *part_i = nullptr;
    // Batched calls: the instance table and call-state staging, kept across calls (grown on
    // demand), and the HIP graph of the last captured call with the launch structure it was
    // captured for (replayed while a call has the same structure).
    InstanceDesc *table = nullptr;
    size_t table_cap = 0;
    BatchStage *stages = nullptr;
    size_t stages_cap = 0;
    int32_t *stage = nullptr;
    size_t stage_cap = 0;
    int32_t *rounds = nullptr;
    size_t rounds_cap = 0;
    int32_t *out = nullptr;
    size_t out_cap = 0;
    hipGraphExec_t exec = nullptr;
    std::vector<int64_t> exec_key;
};
// The largest instance of a batch.
struct MultiSize {
    int64_t n = 0, m = 0, nclaim = 0, nreach = 0, nsrc = 0;
    bool lt = false, forest = true;
    void add(const imin_graph *g);
};
int multi_alloc(MultiScratch &ms, int num_cus, const MultiSize &size, uint32_t cap,
                int32_t max_inst, hipStream_t stream);
void multi_free(MultiScratch &ms);
// One round of every instance of the device table inst[0..ninst) (sample indices
// [0, total), keys seed + round, greedy round step + round): for GreedyReplace instances in
// their replacement pass (gr) the unblocking of that round's slot, then the wavefront-level
// kernels, the workgroup kernels for the samples they hand over, then (select) each
// instance's greedy choice, applied (launch_batch_argmax; instances that end their run add
// one to ms.ctrl[9]). Nothing waits for the host. D is cleared first.
int multi_round(MultiScratch &ms, const InstanceDesc *inst, int32_t ninst, uint32_t total,
                uint32_t round, const imin_launch &shape, int num_cus, bool select, bool gr,
                bool lt, hipStream_t stream);
// GreedyReplace's first-phase candidates CB = out-neighbours of the seeds that are not
// seeds, as a bitmap over g's vertices; returns |CB|.
int32_t gr_candidates(const imin_graph *g, const std::vector<int32_t> &seeds,
                      const std::vector<uint32_t> &inelig, std::vector<uint32_t> &cand);
// The error words of the last rounds (0 when every sample was counted).
int multi_errors(MultiScratch &ms, uint32_t *wave_err, uint32_t *wg_err, hipStream_t stream);

}  // namespace host
}  // namespace imin
