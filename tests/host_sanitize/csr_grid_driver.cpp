// The grid of the scalar path's launch, checked without a GPU: every launch stays below 2^32 threads, and its workgroups
// cover every (tier, slice, block) exactly once.  Built and run by tests/test_host_sanitize.py.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "csr_grid.hpp"

using namespace hcspmm;

static int fail(const char* what, long long a, long long b) { std::fprintf(stderr, "FAILED: %s (%lld, %lld)\n", what, a, b); return 1; }

// the kernel's own walk over the tiers (spmm_csr_kernels.hip, k_csr)
static int check_cover(const CsrGrid& g, int group, int64_t n_segs, int64_t n_mid, int64_t n_items)
{
    const uint32_t per[3] = {g.seg_blocks, g.mid_blocks, g.short_blocks};
    const int run[3] = {-1, g.run_mid, g.run};
    const int64_t need[3] = {n_segs, (n_mid + 3) / 4, (n_items + 256 / group * g.rows_per_group - 1) / (256 / group * g.rows_per_group)};
    std::vector<std::vector<uint8_t>> seen(3);
    for (int t = 0; t < 3; ++t) seen[t].assign((size_t)per[t] * g.n_slices, 0);
    for (int64_t id = 0; id < g.blocks(); ++id) {
        uint32_t b = (uint32_t)id;
        int t = 0;
        while (b >= per[t] * (uint32_t)g.n_slices) b -= per[t] * (uint32_t)g.n_slices, ++t;
        int slice;
        const uint32_t blk = csr_block((uint32_t)id, b, per[t], run[t], g.n_slices, slice);
        if (slice < 0 || slice >= g.n_slices || blk >= per[t]) return fail("block outside its tier", id, blk);
        if (seen[t][(size_t)slice * per[t] + blk]++) return fail("block taken twice", id, blk);
    }
    for (int t = 0; t < 3; ++t)
        if (per[t] < need[t]) return fail("tier too small", per[t], need[t]);
    return 0;
}

int main()
{
    for (int n_slices : {1, 2, 3, 4, 5, 8, 16})
        for (int run : {-1, 0, 5})
            for (int64_t n_items : {0ll, 1ll, 16ll, 17ll, 16383ll, 16384ll, 16400ll, 70001ll})
                for (int64_t n_mid : {0ll, 3ll, 4095ll, 4097ll, 9000ll})
                    for (int64_t n_segs : {0ll, 1ll, 9ll, 1031ll})
                        for (int rpg : {1, 3, 8, 16}) {
                            const int group = rpg == 16 || n_segs == 9 ? 16 : 8;
                            const CsrGrid g = csr_grid(n_segs, n_mid, n_items, 64 * n_slices, n_slices, 64, run, group, rpg);
                            if (g.n_slices != n_slices || g.rows_per_group != rpg) return fail("changed without need", n_slices, rpg);
                            if (check_cover(g, group, n_segs, n_mid, n_items)) return 1;
                        }
    // launches that have to be thinned out: 34 M rows in eight slices of 64 columns, rows of a wave each, 2^31 - 1 rows
    struct Big { int64_t segs, mid, items; int32_t d, n_slices, slice_w; };
    for (const Big& c : {Big{0, 0, 34000000, 512, 8, 64}, Big{0, 0, 34000000, 256, 4, 64}, Big{100, 14000000, 0, 1024, 32, 32},
                         Big{1000000, 8000000, 500000000, 1 << 20, 1 << 15, 32}, Big{0, 0, 2147483647, 1, 1, 1},
                         Big{2097152, 16777215, 2130706432, 128, 4, 32}, Big{3, 5, 1 << 28, 96, 3, 32}}) {
        const int group = c.slice_w == 32 ? 8 : 16;
        const CsrGrid g = csr_grid(c.segs, c.mid, c.items, c.d, c.n_slices, c.slice_w, 5, group);
        const int64_t blocks = g.blocks();
        if (blocks > kMaxBlocks) return fail("launch too large", blocks, c.items);
        if ((int64_t)g.slice_w * g.n_slices < c.d || (int64_t)g.slice_w * (g.n_slices - 1) >= c.d) return fail("slices do not cover the width", g.slice_w, c.d);
        if (g.rows_per_group < 1 || g.rows_per_group > group) return fail("rows per group", g.rows_per_group, 0);
        if (blocks <= 20000000 && check_cover(g, group, c.segs, c.mid, c.items)) return 1;
    }
    std::printf("csr grid driver: ok\n");
    return 0;
}
