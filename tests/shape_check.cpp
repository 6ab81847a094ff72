// Launch shapes of the LDS-claim kernel, on the host: the bitmap and the fixed part fit a
// workgroup's LDS, the workgroups fit the compute unit, and a graph that is taken keeps at least
// 512 threads at work on it. Built without device code.
#include "tree.hip"

#include <cstdio>

using namespace imin;

int main()
{
    long taken = 0;
    for (int64_t nclaim = 0; nclaim <= 1400000; nclaim += nclaim < 2000 ? 1 : 63)
        for (int reach_only = 0; reach_only < 2; ++reach_only)
            for (int64_t theta : {1, 300, 700, 2000, 10000, 1000000})
                for (int64_t seed_edges : {-1, 40, 1000, 50000})
                for (int32_t block : {0, 64, 128, 256, 512, 1024}) {
                    TreeShape s;
                    TreeFit f;
                    f.nclaim = nclaim;
                    f.nreach = nclaim + nclaim / 2;
                    f.reach_only = reach_only != 0;
                    f.theta = theta;
                    f.num_cus = 256;
                    f.seed_edges = seed_edges;
                    f.block = block;
                    if (!tree_shape(f, s)) {
                        if (block == 0 && nclaim <= 1200000) return std::printf("refused %ld\n", (long)nclaim), 1;
                        continue;
                    }
                    ++taken;
                    // many-instance launches, whose kernel has two sizes
                    if (seed_edges < 0 && !reach_only && !block && theta == 1000000 &&
                        f.nreach > (1 << 17) && s.block != 512 && s.block != 1024)
                        return std::printf("nclaim %ld: %d threads\n", (long)nclaim, s.block), 1;
                    const size_t head = s.block == 64    ? head_bytes<64>()
                                        : s.block == 128 ? head_bytes<128>()
                                        : s.block == 256 ? head_bytes<256>()
                                        : s.block == 512 ? head_bytes<512>()
                                                         : head_bytes<1024>();
                    const int64_t words = (nclaim + 31) / 32;
                    if (s.bm_words < words || head + 4 * (size_t)words > s.lds ||
                        (size_t)s.per_cu * s.lds > kTreeLds || s.per_cu < 1 ||
                        s.per_cu * s.block > 256 * kTreeWaves || (block && s.block != block) ||
                        (!block && s.per_cu * s.block < 512))
                        return std::printf("nclaim %ld theta %ld: %d x %d threads, %u bytes\n", (long)nclaim,
                                           (long)theta, s.per_cu, s.block, s.lds), 1;
                }
    std::printf("shapes ok: %ld\n", taken);
    return 0;
}
