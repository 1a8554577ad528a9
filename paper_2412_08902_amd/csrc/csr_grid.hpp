// The grid of the scalar path's launch (spmm_csr_kernels.hip): how many workgroups each tier gets per column slice, and
// which part of the work a workgroup is.  Plain C++, so that the mapping can be checked without a GPU.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define HC_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define HC_HOST_DEVICE inline
#endif

namespace hcspmm {

constexpr int64_t kMaxBlocks = ((int64_t)1 << 24) - 1;   // workgroups of 256 threads in a launch: fewer than 2^32 threads

struct CsrGrid {
    uint32_t seg_blocks, mid_blocks, short_blocks;  // workgroups of each tier and slice, padded (surplus ones exit at once)
    int32_t rows_per_group;
    int32_t run, run_mid;              // log2 of the workgroups per XCD-local run of the short and mid tiers (-1: plain order)
    int32_t n_slices, slice_w;         // column slices
    HC_HOST_DEVICE int64_t blocks() const { return ((int64_t)seg_blocks + mid_blocks + short_blocks) * n_slices; }
};

// Tiers: n_segs segments of long rows, n_mid rows of a wave each (four to a workgroup), n_items short rows of a group each.
// XCD-local runs (see csr_block): tiers of at least 1024 workgroups are padded to whole rounds of runs of 2^run workgroups
// over the XCDs that share a slice.  A group (of 8 or 16 lanes) takes one row -- what one after the other adds is only the chain of its loads --
// unless the launch would have more threads than a launch may: then first more rows to a group (at most as many as it has
// lanes; the kernel's wide forms walk them one after the other), then wider slices.
inline CsrGrid csr_grid(int64_t n_segs, int64_t n_mid, int64_t n_items, int32_t d, int32_t n_slices, int32_t slice_w, int run,
                        int group, int rows_per_group = 1)
{
    CsrGrid g{};
    g.rows_per_group = rows_per_group;
    g.n_slices = n_slices;
    g.slice_w = slice_w;
    for (;;) {
        const bool owned = g.n_slices == 2 || g.n_slices == 4 || g.n_slices == 8;
        const int64_t nsub = owned ? 8 / g.n_slices : 8;
        auto padded = [&](int64_t n, int32_t& r) {
            r = n < 1024 ? -1 : run;
            const int64_t unit = nsub << (r > 0 ? r : 0);
            return r >= 0 || owned ? (n + unit - 1) / unit * unit : n;
        };
        const int64_t per_block = (int64_t)(256 / group) * g.rows_per_group;
        const int64_t segs = owned ? (n_segs + nsub - 1) / nsub * nsub : n_segs;
        const int64_t mid = padded((n_mid + 3) / 4, g.run_mid), shorts = padded((n_items + per_block - 1) / per_block, g.run);
        if ((segs + mid + shorts) * g.n_slices <= kMaxBlocks || (g.n_slices == 1 && g.rows_per_group == group)) {
            g.seg_blocks = (uint32_t)segs; g.mid_blocks = (uint32_t)mid; g.short_blocks = (uint32_t)shorts;
            return g;
        }
        if (shorts > 0 && g.rows_per_group < group) {
            g.rows_per_group = 2 * g.rows_per_group < group ? 2 * g.rows_per_group : group;
        } else if (g.n_slices > 1) {
            g.slice_w = 2 * (int64_t)g.slice_w < d ? 2 * g.slice_w : d;
            g.n_slices = (int32_t)(((int64_t)d + g.slice_w - 1) / g.slice_w);
        } else {
            g.rows_per_group = group;
        }
    }
}

// Block b of a tier of `blocks` workgroups per slice, of the launch's workgroup `id` -> (slice, block within the tier).
// Workgroups go to the eight XCDs round-robin by their linear id, and each XCD has an L2 of its own.
//  * The tier's blocks are handed out in runs of 2^run consecutive ones that stay on one XCD: neighbouring rows -- which
//    share columns in graphs with any locality -- meet in one L2 close in time, while all XCDs still advance through the
//    matrix side by side (rows sorted by degree stay balanced).
//  * With 2, 4 or 8 column slices XCD x works on slice x % n_slices only, so that its L2 holds rows of ONE slice.
//  * Other slice counts take the slices one after the other.
HC_HOST_DEVICE uint32_t csr_block(uint32_t id, uint32_t b, uint32_t blocks, int run, int n_slices, int& slice)
{
    const uint32_t x = id & 7;
    slice = 0;
    uint32_t nsub = 8, sub = x;
    if (n_slices > 1) {
        if (n_slices == 2 || n_slices == 4 || n_slices == 8) {
            nsub = 8 / n_slices;
            slice = (int)(x & (n_slices - 1));
            sub = x / n_slices;
            run = run > 0 ? run : 0;
        } else {
            slice = (int)(b / blocks);
            b -= (uint32_t)slice * blocks;
        }
    }
    if (run < 0) return b;
    const uint32_t q = b >> 3;
    return ((((q >> run) * nsub) + sub) << run) + (q & ((1u << run) - 1));
}

}  // namespace hcspmm
