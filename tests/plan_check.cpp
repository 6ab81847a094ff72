// The no-allocation call's scratch plans, on the host: over random graphs, what the layout of the
// kernel of large claim sets accepts, the LDS-claim kernel's accepts too, with every array inside
// the scratch and apart from the others. Built without device code.
#include "noalloc.hip"

#include <cstdio>
#include <random>

namespace {

// The arrays of a call that come before the slots'.
Carve call_arrays(const imin_graph &g, uint32_t theta, int32_t nS, bool blocked)
{
    Carve c{reinterpret_cast<unsigned char *>(size_t(1) << 32)};
    c.take<uint32_t>((size_t)g.words);
    c.take<int32_t>((size_t)nS);
    c.take<int32_t>((size_t)nS);
    c.take<uint32_t>(1);
    if (blocked) c.take<uint8_t>((size_t)g.n);
    c.take<uint32_t>(theta);
    c.take<uint32_t>(theta);
    return c;
}

// The layout of the kernel that claims in device memory (linear threshold: without row ranges).
bool device_claims_fit(Carve c, const imin_graph &g)
{
    const int64_t n = g.n, lcap = n + 1, xmax = (int64_t)g.m + 1, xcap = extra_cap(n, g.m);
    auto slots = [&](size_t count, int64_t extra) {
        c.take<unsigned long long>(count * (size_t)n);
        c.take<imin::LocalVtx>(count * (size_t)lcap);
        c.take<int32_t>(count * (size_t)(lcap + 1));
        c.take<int2>(count * (size_t)std::max<int64_t>(extra, 1));
        c.take<uint32_t>(count);
        c.take<uint32_t>(count);
        if (g.model == IMIN_IC) c.take<int2>(count * (size_t)lcap);
        return c.fits;
    };
    return (xcap >= xmax || slots(2, xmax)) && slots(1, xcap);
}

}  // namespace

int main()
{
    std::mt19937_64 rng(1);
    std::uniform_real_distribution<double> u(0.0, 1.0);
    auto log_int = [&](double lo, double hi) { return (int64_t)std::exp(std::log(lo) + u(rng) * std::log(hi / lo)); };
    long accepted = 0, more = 0, one_large = 0, few_extra = 0;
    for (long i = 0; i < 400000; ++i) {
        imin_graph g;
        g.model = u(rng) < 0.7 ? IMIN_IC : IMIN_LT;
        g.num_cus = 256;
        g.n = (int32_t)log_int(1, 1.2e7);
        // some graphs with as many edges as just fit two large slots
        g.m = u(rng) < 0.5 ? (int32_t)log_int(1, 3e7)
                           : (int32_t)std::max(1.0, (268435456.0 - 120.0 * g.n) / 16.0 * (0.97 + 0.04 * u(rng)));
        g.words = (g.n + 31) / 32;
        g.nreach = (int32_t)(std::min(g.n, g.m) * (u(rng) < 0.5 ? 1.0 : u(rng)));
        g.nclaim = std::min((int32_t)(g.nreach * u(rng)), g.m / 2);
        const uint32_t theta = (uint32_t)log_int(1, 1e6);
        g.seed_edges = log_int(1, 1e5);
        if (!imin::tree_shape(tree_fit(&g, 1, false), g.shape)) continue;
        const Carve start = call_arrays(g, theta, (int32_t)log_int(1, 1e4), u(rng) < 0.5);
        imin::TreeWs main_tw, big_tw;
        Carve c = start;
        const bool fits = start.fits && carve_tree_call(c, &g, theta, g.shape, main_tw, big_tw);
        const bool before = start.fits && device_claims_fit(start, g);
        if (before && !fits) {
            std::printf("refused: n %d m %d nreach %d nclaim %d theta %u\n", g.n, g.m, g.nreach, g.nclaim, theta);
            return 1;
        }
        accepted += before;
        more += fits && !before;
        if (!fits) continue;
        if (main_tw.slots < 1 || (main_tw.xcap <= g.m && g.model == IMIN_IC && big_tw.slots < 1) ||
            (big_tw.slots > 0 && big_tw.xcap != (int64_t)g.m + 1) || c.used > kScratchBytes) {
            std::printf("bad plan: n %d m %d slots %d + %d\n", g.n, g.m, main_tw.slots, big_tw.slots);
            return 1;
        }
        unsigned char *end = start.base + start.used;
        for (const imin::TreeWs *w : {&big_tw, &main_tw}) {
            if (w->slots == 0) continue;
            if (reinterpret_cast<unsigned char *>(w->planes) < end) {
                std::printf("overlap: n %d m %d\n", g.n, g.m);
                return 1;
            }
            end = reinterpret_cast<unsigned char *>(w->extra + w->slots * w->xcap);
        }
        if (end > start.base + kScratchBytes) {
            std::printf("beyond the scratch: n %d m %d\n", g.n, g.m);
            return 1;
        }
        one_large += big_tw.slots == 1;
        few_extra += g.model == IMIN_IC && main_tw.xcap < extra_cap(g.n, g.m);
    }
    std::printf("plans ok: accepted %ld, more %ld, one large slot %ld, fewer extra edges %ld\n", accepted,
                more, one_large, few_extra);
    return accepted > 0 && one_large > 0 && few_extra > 0 ? 0 : 1;
}
