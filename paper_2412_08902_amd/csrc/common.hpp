// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "hcspmm.h"

namespace hcspmm {

constexpr int kH = 16;                 // rows per window (Section IV-A: the minimum hybrid unit)
// launch guard of the hybrid routing: a path with fewer non-zeros than kGuardNnz and less than
// 1/kGuardShare of the matrix gives its windows to the other path
constexpr int64_t kGuardNnz = 1 << 18;
constexpr int64_t kGuardShare = 8;

// ---- preprocessing -----------------------------------------------------------------------------
constexpr int kCountTinyCap = 1024;    // windows with at most this many non-zeros are counted in an 8 KB LDS hash set
constexpr int kUniqueSmallCap = 4096;  // windows with at most this many non-zeros are condensed by an LDS sort
constexpr int kCountMidCap = 16384;    // windows up to this many non-zeros are counted with an LDS hash set (128 KB)
constexpr int kBitmapWords = 32768;    // LDS bitmap (1 Mi columns per pass) used to condense larger windows
constexpr int kEcolLdsCap = 4096;      // distinct-column lists up to this length are searched from LDS

// ---- matrix path -------------------------------------------------------------------------------
constexpr int kMfmaSmallMaxCols = 256; // windows with more condensed columns go to a workgroup-per-window kernel
constexpr int kMfmaMidMaxCols = 1024;  // ... with the small LDS chunk up to here, the large chunk beyond
constexpr int kKcMid = 256;            // condensed columns staged per workgroup and chunk, medium windows
constexpr int kKcBig = 1024;           // condensed columns staged per workgroup and chunk, wide windows
constexpr int kSliceCols = 4096;       // condensed columns per workgroup; wider windows are cut into slices

// ---- scalar path -------------------------------------------------------------------------------
constexpr int kMidRow = 128;           // rows with more non-zeros than this get a whole wave
// On a matrix of few rows the longest chain of dependent loads is what a call takes, so a wave takes rows over earlier
// (30,000 rows, fp32, 64 columns: 16.4 -> 14.9 us; 16,000 rows, bf16, 128 columns: 11.1 -> 8.0 us); large ones lose 3-7 %.
constexpr int kMidRowSmall = 64, kMidRowFewRows = 65536;
constexpr int kFusedMidRow = 256;      // with the update stage fused in, rows up to this length stay in the workgroup's tile
constexpr int kLongRow = 1024;         // rows with more non-zeros than this are cut into workgroup-sized segments
// ... from 256 non-zeros on where rows have fewer than 100 on average: a wave that walks 1000 non-zeros outlasts everything
// else there (rows cut from 1024 / from 256 non-zeros on, 64 columns, bf16: 320 rows of 20 with some of 1000: 13.7 / 5.6 us,
// 2,000 of 60 with some of 400: 7.7 / 5.0 us, 16,000 of 60: 16.5 / 10.6 us, 65,000 of 20: 28.2 / 17.7 us, 169,000 of 20: 45.1 /
// 44.4 us; 128 columns, fp32: 9.7 / 5.0 us for the first, 29.2 / 29.3, 52.4 / 51.5 and 162 / 162 us; 8 lanes to a row, 32
// columns: 200,000 rows of 10: 42 / 29.5 us, 350,000: 56 / 50.6 us).  On more rows the long ones are hidden: level within 2 %
// to 2.4 M rows.  A matrix of a handful of rows keeps the plain tiers.  256 threads per row only add their reduction where
// long rows are many (30,000 of 200: 183 -> 192 us).
constexpr int kLongRowSparse = 256;
constexpr int64_t kLongRowDegree = 100;
constexpr int32_t kLongRowFewRows = 256;
constexpr int kSegLen = 2048;          // non-zeros per segment of a long row

struct Segment { int32_t row, k_begin, k_end, slot; };    // slot < 0: writes Y directly
struct MultiRow { int32_t row, first_slot, n_slots, pad; };
// everything the wave-per-window matrix kernel needs to start on a window, in one 32-byte read
// one workgroup's share of a matrix-path window: condensed columns [kc_begin, kc_end); slot < 0: writes Y
struct WgSlice { int32_t w, kc_begin, kc_end, slot; };
struct WinDesc { int32_t w, s, e, nc; int64_t wp; int64_t pad; };
// a run of up to kRunWindows consecutive entries of the matrix path's window list whose column lists were merged
struct RunDesc { int64_t up; int32_t first, nw, nu, n_slices, slot0, pad; };   // union at ucols[up .. up + nu)
// one workgroup's share of a run: union positions [u_begin, u_end) of the list at ucols[up ..], q-th of the run's
// n_slices slices; nw windows; partial tiles (n_slices > 1) at slot0 + wave * n_slices + q
struct RunSlice { int64_t up; int32_t run, u_begin, u_end, q, nw, n_slices, slot0, pad[3]; };
// the window a wave of a slice's workgroup owns (waves beyond the run's last window repeat its first)
struct RunWin { int64_t wp; int32_t w, nc, k_last, pad; };
constexpr int kRunWindows = 4;

void set_error(const char* fmt, ...);

// Experiment knobs (HCSPMM_TUNE_* environment variables; not part of the ABI), read ONCE per process on first use.
// A value of -1 means "not set": the built-in choice applies.
struct Tune {
    int mid_row, long_row, slice_cols, serial, xcd_chunk, rpg, tiles_per_wave, runs, run_slice, side_nnz, bands;
};
const Tune& tune();

#define HC_HIP(call)                                                                               \
    do {                                                                                           \
        hipError_t e_ = (call);                                                                    \
        if (e_ != hipSuccess) {                                                                    \
            ::hcspmm::set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), __FILE__, __LINE__); \
            return HCSPMM_EHIP;                                                                    \
        }                                                                                          \
    } while (0)

// Exclusive prefix sum of n int32 values into n+1 int64 values (out[n] = total).  `scratch` holds
// at least scan_scratch_elems(n) int64.  Enqueued on `stream`.
size_t scan_scratch_elems(int64_t n);
hipError_t exclusive_scan_i32_i64(const int32_t* in, int64_t n, int64_t* out, int64_t* scratch, hipStream_t stream);
// up to kScanMaxArrays arrays of one length in one pass: out[a] (n + 1 entries; may be null when only the total is
// wanted) and totals_dev[a] (device, may be null) for every array a; scratch holds scan_multi_scratch_elems(n) values
constexpr int kScanMaxArrays = 8;
struct ScanMulti { const int32_t* in[kScanMaxArrays]; int64_t* out[kScanMaxArrays]; int k; };
size_t scan_multi_scratch_elems(int64_t n);
hipError_t exclusive_scan_multi(const ScanMulti& m, int64_t n, int64_t* totals_dev, int64_t* scratch, hipStream_t stream);

// ---- preparation (prepare_kernels.hip): CSR arrays -> window features, routes, row tables -------
struct PrepTotals {
    int64_t total_ncols, nnz_mfma, wide_cols /* columns of wide matrix-path windows */, mfma_cols /* of all of them */, nnz_long, n_slots;
    int32_t n_mfma, n_mfma_small, n_mfma_mid, n_mfma_big, n_short, n_mid, n_rest, n_multi, n_segs;
    int32_t all_scalar;                   // every window runs on the scalar path, 2: in column panels (see scalar_form)
    int32_t sample_distinct;              // see sample_share
    int32_t n_big_list, n_huge_list;      // windows above kUniqueSmallCap / kCountMidCap non-zeros
    int32_t err;                          // 1 rowptr[0], 2 rowptr[n_rows], 4 decreasing rowptr, 8 column out of range
};
constexpr int kPrepCtl = 16;
constexpr int32_t kSampleSlices = 16384, kSamplePanels = 65536;   // non-zeros per stretch of the sample (see build_plan)
struct Prep {
    int32_t n_rows, n_cols, W, n_tiles;
    int64_t nnz;
    const int32_t *rowptr, *colind;
    int32_t* ctl;                         // kPrepCtl zeros: [0] errors, [1] [2] lengths of big_list, huge_list, [3] of count_1k,
                                          // [4] [5] of count_mid, count_huge, [6] unsorted rows, [7] all scalar, [8] sample
    int32_t *big_list, *huge_list;        // every window of the two classes
    int32_t *count_1k, *count_mid, *count_huge, *n_count_mid, *n_count_huge;   // windows whose columns are still to be counted
    int32_t* on_matrix;                   // set by launch_prep: non-zeros that the selector sends to the matrix path, per window
    const int32_t* touched;               // windows to count (null: all)
    const int32_t* old_ncols;             // counts carried over for the others
    int32_t features;                     // distinct columns are wanted
    int32_t sample_len;                   // non-zeros per stretch of the sample, nnz at most (0: no sample)
    int32_t panels_from;                  // panels are asked for: from this percentage of distinct columns in the sample on (0: not)
    int32_t scalar_exec;                  // every window may run on the scalar path (see scalar_form)
    int32_t big_takes_1k;                 // set by launch_prep
    int32_t mode;
    long long c0, c1, c2;
    int32_t mid_row, long_row, fused_mid_row;
    int32_t *ncols, *nnzw;
    uint8_t* route;
    int64_t* wptr;
    unsigned long long *wt, *rt;          // sums per tile of 64 windows: of its windows, of its rows (see prep_bind_sums)
    unsigned long long *wg, *rg;          // ... and per group of tiles (null: a matrix of few tiles)
    int32_t *short_rows, *mid_rows, *rest_rows;   // row tables to fill (null: skip)
    Segment* segs;
    MultiRow* multi;
    PrepTotals* out;                      // host or device memory (null: skip)
};
// Column panels of the scalar path (see run_spmm): where every row enters each panel, and each panel's row tables.
constexpr int kMaxPanels = 16, kPanelRowBytes = 128;            // panels for X rows of at least that many bytes
struct PanelTotals { int64_t nnz, n_slots; int32_t n_mid, n_segs, n_multi, pad; };
struct PanelArgs {
    int32_t n_rows, n_cols, n_panels, n_tiles, mid_row, long_row;
    const int32_t *rowptr, *colind;
    int32_t* split;                       // n_panels - 1 arrays of n_rows: first non-zero at or beyond the panel's end
    unsigned long long* sums;             // panel_sum_words: 3 per panel and tile, and per panel and group of tiles
    unsigned long long* groups;           // set by launch_panels, as n_groups
    int32_t n_groups;
    int64_t cap_mid, cap_segs, cap_multi; // entries per panel of
    int32_t* mid_rows;
    Segment* segs;
    MultiRow* multi;
    PanelTotals* out;                     // n_panels
};
hipError_t launch_panels(const PanelArgs& p, hipStream_t s);
size_t prep_tile_count(int32_t W);
size_t prep_tile_words(int32_t W);        // 64-bit words of all sums of a preparation
void prep_bind_sums(Prep& p, unsigned long long* words);       // sets n_tiles, wt, rt, wg and rg (from W)
size_t panel_sum_words(int32_t n_panels, int32_t n_tiles);
double sample_share(const Prep& p, int32_t distinct);          // distinct columns per non-zero of the sampled stretches (1: no sample)
size_t prep_zeros(const Prep& p, int32_t n_touched);            // bytes of p.wt that launch_prep expects to be zeros
hipError_t launch_prep(const Prep& p, int32_t n_touched, hipStream_t s);
hipError_t launch_prep_fill(const Prep& p, hipStream_t s);      // another pass over the row tables
hipError_t launch_prep_windows(const Prep& p, int32_t* mfma, int32_t* small, int32_t* mid, int32_t* big, hipStream_t s);

// ---- preprocessing launchers (prepare_kernels.hip) ---------------------------------------------
hipError_t launch_window_nnz(int32_t W, int32_t n_rows, const int32_t* rowptr, int32_t* nnzw, int32_t* big_list,
                             int32_t* big_count, hipStream_t s);
// sorted distinct-column lists (route: null = every window, else only windows with route != 0)
hipError_t launch_unique_small(int32_t W, int32_t n_rows, const int32_t* rowptr, const int32_t* colind,
                               int32_t* tmp_cols, int32_t* ncols, const uint8_t* route, hipStream_t s);
hipError_t launch_unique_big(int32_t n_big, const int32_t* big_list, int32_t n_rows, int32_t n_cols,
                             const int32_t* rowptr, const int32_t* colind, int32_t* tmp_cols, int32_t* ncols,
                             const uint8_t* route, hipStream_t s);
// incremental preparation: which matrix-path windows keep the previous plan's condensed structure, and its copy
hipError_t launch_carry_mask(int32_t W, const uint8_t* old_route, const uint8_t* route, int32_t n_touched,
                             const int32_t* touched, uint8_t* carried, uint8_t* todo, hipStream_t s);
hipError_t launch_carry_copy(int32_t W, int32_t n_rows, const uint8_t* carried, const int64_t* old_wptr, const int64_t* wptr,
                             const int32_t* old_wcols, int32_t* wcols, const int64_t* old_start, const int32_t* rowptr,
                             const int32_t* old_erc, int32_t* erc, hipStream_t s);
hipError_t launch_ecol(int32_t W, int32_t n_rows, const int32_t* rowptr, const int32_t* colind,
                       const int32_t* tmp_cols, const int32_t* ncols, const int64_t* wptr, int32_t* wcols,
                       int32_t* erc, int32_t* unsorted_flag, const uint8_t* route, int want,
                       int32_t skip_above /* leave windows with more non-zeros alone */, hipStream_t s);
// sorted list and condensed positions of the listed matrix-path windows by bitmap ranks (no search)
hipError_t launch_condense_rank(int32_t n_list, const int32_t* list, int32_t n_rows, const int32_t* rowptr,
                                const int32_t* colind, const uint8_t* route, const int64_t* wptr, int32_t* wcols,
                                int32_t* erc, int32_t* unsorted_flag, hipStream_t s);
constexpr int64_t kRankMaxCols = (int64_t)8 << 19;   // beyond this many columns a window's bitmap passes cost more than searching
hipError_t launch_build_desc(int32_t n_list, const int32_t* win_list, int32_t n_rows, const int32_t* rowptr,
                             const int32_t* ncols, const int64_t* wptr, WinDesc* desc, hipStream_t s);
hipError_t launch_slice_count(int32_t n_list, const int32_t* win_list, const int32_t* ncols, int32_t slice_cols,
                              int32_t* n_slices, int32_t* f_multi, int32_t* n_slots, hipStream_t s);
hipError_t launch_slice_fill(int32_t n_list, const int32_t* win_list, const int32_t* ncols, int32_t slice_cols,
                             const int64_t* slice_pos, const int64_t* multi_pos, const int64_t* slot_pos,
                             WgSlice* slices, MultiRow* multi, hipStream_t s);

// ---- compute launchers -------------------------------------------------------------------------
struct SpmmArgs {
    int32_t n_rows;
    int32_t n_cols;       // rows of X
    const int32_t* rowptr;
    const int32_t* rowend;    // null, or a column panel's share of the rows: row i is [rowptr[i], rowend[i])
    const int32_t* colind;
    const float* vals;
    const void* X;
    int64_t ldx;
    int32_t d;
    int32_t x_dtype;
    float* Y;             // element type y_dtype (fp32 unless the caller asked for a 16-bit output); ldy in elements
    int64_t ldy;
    int32_t relu;
    int32_t y_dtype;
    const float* acc;     // scalar path: fp32 rows (pitch ldacc) added to the result before the activation and the store; may be Y
    int64_t ldacc;
    const uint2* x_mask;  // scalar path, where csr_mask_usable says so: which elements of X count (launch_relu_bits), the others are 0
};

// Update stage of the aggregate-then-update layer: Y = act(Z W) for aggregated rows Z (Section V-A).
struct UpdateArgs {
    const float* W;       // d_in x d_out, fp32
    int64_t ldw;
    int32_t d_out;
    float* Y;             // n_rows x d_out
    int64_t ldy;
    int32_t relu;
    int32_t keep_z;       // also store every aggregated row to the workspace (a.Y), not only the rows finished later
    const float* mask;    // optional, n_rows x d_out (pitch ldm): results are stored as 0 where mask <= 0
    int64_t ldm;
    int32_t y_dtype;      // element type of Y
};

#if defined(__HIPCC__)
// fp32 -> 16-bit storage, one rounding to nearest even (the only rounding a 16-bit output adds to the fp32 result);
// two values per call, packed low | high << 16.  The conversions are the hardware's (gfx950 converts to bf16 natively).
typedef float out_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 out_bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 out_f16x2 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t out16_pack(float lo, float hi, int y_dtype)
{
    const out_f32x2 v = {lo, hi};
    if (y_dtype == HCSPMM_BF16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, out_bf16x2));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, out_f16x2));
}

// Stores VEC consecutive results at element offset `off` of an output matrix of element type y_dtype, after the
// optional max(0, .).  The address is aligned for VEC fp32 elements when y_dtype is fp32 and for min(VEC, 4) 16-bit
// elements otherwise (no 16-bit store is wider than 8 bytes).
// BRANCH: without an activation nothing is spent on one.  To select costs three instructions a value with or without, which rows of 16-bit X on the scalar
// path are bound by, one vector to a lane (select / branch, us: communities, 131,072 rows of 20, bf16, 64 columns: 22.5 / 21.8, 65,536 of 13 behind a product: 24.5 / 24.4; power law, 100,000 of
// 7: 14.0 / 13.7; but two vectors, 662,778 of 10, 144: 315.5 / 320.4).  fp32 rows, which need nothing widened, are level or lose (communities, 32 columns: 20.16 / 20.14; power law, 300,000 of 6, 8 columns: 18.97 / 19.10,
// 20,641 of 6, 32 columns and a product: 18.5 / 18.6).  Matrix tiles and the dense products lose too, whose results all wait behind the branch: 299,968 rows of 58, 208 -> 48
// with an activation: 222.7 / 224.3; without one, by the kernel trace, 2,197 x 235 x 224 (k_gemm_split): 13.16 / 13.36, 3,559 x 128 x 112 (k_gemm_f32, the
// shortest of 600): 7.71 / 7.85, 5,625 x 103 x 48: 6.50 / 6.62; large ones level.
template <int VEC, bool BRANCH = false> __device__ inline void out_store(float* __restrict__ Y, int y_dtype, int64_t off, const float (&x)[VEC], int relu)
{
    float y[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) y[i] = BRANCH || !relu ? x[i] : fmaxf(x[i], 0.f);
    if (BRANCH && relu) {
        asm volatile("");                                       // (stays a branch)
#pragma unroll
        for (int i = 0; i < VEC; ++i) y[i] = fmaxf(x[i], 0.f);
    }
    if (y_dtype == HCSPMM_F32) {
        float* __restrict__ p = Y + off;
        if constexpr (VEC == 8) {
            *reinterpret_cast<float4*>(p) = make_float4(y[0], y[1], y[2], y[3]);
            *reinterpret_cast<float4*>(p + 4) = make_float4(y[4], y[5], y[6], y[7]);
        } else if constexpr (VEC == 4) {
            *reinterpret_cast<float4*>(p) = make_float4(y[0], y[1], y[2], y[3]);
        } else if constexpr (VEC == 2) {
            *reinterpret_cast<float2*>(p) = make_float2(y[0], y[1]);
        } else {
            *p = y[0];
        }
    } else {
        unsigned short* __restrict__ p = reinterpret_cast<unsigned short*>(Y) + off;
        if constexpr (VEC >= 4) {
#pragma unroll
            for (int i = 0; i < VEC; i += 4)
                *reinterpret_cast<uint2*>(p + i) = make_uint2(out16_pack(y[i], y[i + 1], y_dtype), out16_pack(y[i + 2], y[i + 3], y_dtype));
        } else if constexpr (VEC == 2) {
            *reinterpret_cast<uint32_t*>(p) = out16_pack(y[0], y[1], y_dtype);
        } else {
            *p = (unsigned short)out16_pack(y[0], 0.f, y_dtype);
        }
    }
}
#endif

// With `upd` the kernels that can keep a 16-row result tile on chip multiply it by W and write
// upd->Y (short rows of the scalar path, wave-per-window tiles of the matrix path); every other
// row goes to a.Y, which then is the aggregation workspace Z, and launch_update_rest finishes it.
bool update_fusable(const SpmmArgs& a);
bool mfma_update_fusable(const SpmmArgs& a);
// what the scalar path's launch knows about its rows beyond the launch tables
struct CsrHints {
    int64_t nnz;          // non-zeros of the scalar-path windows
    int64_t rows;
    bool scattered;       // neighbouring rows are known to share few columns
    int32_t long_row;     // rows with more non-zeros are cut into segments
    bool beside;          // the matrix path runs at the same time on streams of its own
    int64_t entries;      // non-zeros of the matrix, which indices of non-zeros stay below
};
hipError_t launch_csr(const SpmmArgs& a, int32_t n_segs, const Segment* segs, float* partial, int32_t n_mid,
                      const int32_t* mid_rows, int32_t n_items, const int32_t* row_list, const uint8_t* route,
                      int32_t mid_row, const CsrHints& hints, hipStream_t s, const UpdateArgs* upd = nullptr);
bool csr_mask_usable(const SpmmArgs& a, const CsrHints& hints);     // launch_csr may be given a.x_mask
bool csr_panels_usable(const SpmmArgs& a);   // the launch has kernels that add to rows of sums for this shape
hipError_t launch_update_rest(const SpmmArgs& a, int32_t n_rest, const int32_t* rest_rows, const UpdateArgs& upd,
                              hipStream_t s);
hipError_t launch_reduce_partials(const SpmmArgs& a, int32_t n_multi, const MultiRow* multi, const float* partial,
                                  hipStream_t s);
hipError_t launch_mfma_small(const SpmmArgs& a, int32_t n_list, const WinDesc* desc, const int32_t* wcols,
                             const int32_t* erc, hipStream_t s, const UpdateArgs* upd = nullptr);
hipError_t launch_mfma_wg(const SpmmArgs& a, int32_t n_list, const WgSlice* slices, const int32_t* ncols,
                          const int64_t* wptr, const int32_t* wcols, const int32_t* erc, int rows_sorted,
                          const int32_t* slice_rows, float* tile_partial, bool wide, hipStream_t s);
hipError_t launch_slice_rows(int32_t n_slices, const WgSlice* slices, int32_t n_rows, const int32_t* rowptr,
                             const int32_t* erc, int32_t* slice_rows, hipStream_t s);
// bare gather of X rows by an index stream (measurement aid)
int64_t probe_gather_blocks(int64_t n, int32_t d);
hipError_t launch_probe_gather(const int32_t* index, int64_t n, const float* X, int64_t ldx, int32_t d, int32_t n_rows_x,
                               float* out, hipStream_t s);
bool mfma_shape_supported(const SpmmArgs& a);
int mfma_walks(const void* base, int64_t ld, int32_t d);     // launches over the windows for fp32 rows of d columns
bool mfma_run_shape_supported(const SpmmArgs& a);
hipError_t launch_mfma_run(const SpmmArgs& a, int32_t n_slices, const RunSlice* slices, const RunWin* wins,
                           const int32_t* ucols, const int32_t* wslot, const int32_t* erc, float* tile_partial, hipStream_t s);
hipError_t launch_run_wins(int32_t n_slices, const RunSlice* slices, const RunDesc* runs, const int32_t* win_list,
                           const int32_t* ncols, const int64_t* wptr, int32_t n_rows, const int32_t* rowptr, RunWin* wins,
                           hipStream_t s);
// union column list of every run and the position of each window column in it (prepare)
hipError_t launch_run_union(int32_t n_runs, const int32_t* win_list, int32_t n_list, const int32_t* ncols,
                            const int64_t* wptr, const int32_t* wcols, int32_t* ucols, int32_t* wslot, RunDesc* runs,
                            hipStream_t s);
constexpr int kRunMinSlice = 2048;     // union columns per workgroup slice of a run, at least
constexpr int kRunTargetSlices = 4096; // ... and about this many slices over all runs of a large matrix
hipError_t launch_reduce_tiles(const SpmmArgs& a, int32_t n_multi, const MultiRow* multi, const float* tile_partial,
                               hipStream_t s);
// T = X W; with a mask (m x n, pitch ldm) T is stored as 0 where it is not positive
hipError_t launch_gemm_f32(int64_t m, int32_t k, int32_t n, const float* X, int64_t ldx, const float* W, int64_t ldw,
                           float* T, int64_t ldt, const float* mask, int64_t ldm, hipStream_t s);
// T = X W in fp32 for X of any element type; 16-bit X needs rows and a base on whole 4-byte words (gemm_x16_usable)
bool gemm_x16_usable(const void* X, int64_t ldx);
hipError_t launch_gemm_x(int64_t m, int32_t k, int32_t n, const void* X, int64_t ldx, int32_t x_dtype, const float* W, int64_t ldw,
                         float* T, int64_t ldt, hipStream_t s);
// backward pass (Eq. 3): dW = X^T S over row spans, activation mask, transpose of W
int32_t gemm_tn_spans(int64_t n_rows, int32_t d_in, int32_t d);
hipError_t launch_gemm_tn(int64_t n_rows, const float* X, int64_t ldx, int32_t d_in, const float* S, int64_t lds_,
                          int32_t d, float* dW, int64_t lddw, float* partial, hipStream_t s);
bool gemm_grad_usable(int64_t n_rows, int64_t ldx, int32_t d_in, int32_t d);
hipError_t launch_gemm_grad(int64_t n_rows, const float* X, int64_t ldx, int32_t d_in, const float* S, int64_t lds_, int32_t d,
                            const float* W, int64_t ldw, float* dX, int64_t lddx, float* dW, int64_t lddw, float* partial, hipStream_t s);
bool relu_bits_usable(int32_t d, const float* Yf, int64_t ldy);
hipError_t launch_relu_bits(int64_t n, int32_t d, const float* Yf, int64_t ldy, uint2* bits, hipStream_t s);   // bits: [ceil(d / 64)][n]
hipError_t launch_relu_mask(int64_t n, int32_t d, const float* G, int64_t ldg, const float* Yf, int64_t ldy, float* Gm,
                            int64_t ldo, hipStream_t s);
hipError_t launch_transpose(int32_t rows, int32_t cols, const float* W, int64_t ldw, float* Wt, hipStream_t s);
// same product with the output stored as t_dtype (fp32, or bf16 / fp16 rounded from the fp32 accumulators).  done_route,
// done_cols: rows of windows that the wave-per-window matrix kernel owns (route != 0, at most kMfmaSmallMaxCols columns) are
// left alone.
hipError_t launch_gemm_f32_out(int64_t m, int32_t k, int32_t n, const float* X, int64_t ldx, const float* W, int64_t ldw,
                               void* T, int64_t ldt, int32_t t_dtype, int relu, hipStream_t s,
                               const uint8_t* done_route = nullptr, const int32_t* done_cols = nullptr,
                               const float* mask = nullptr, int64_t ldm = 0);

}  // namespace hcspmm

struct BlockCache;
struct hcspmm_plan {
    int32_t H, n_rows, n_cols, W;
    int64_t nnz;
    int device;
    hcspmm_options opt;
    int64_t coef[3];
    // borrowed
    const int32_t* rowptr;
    const int32_t* colind;
    const float* vals;
    // owned, canonical
    int32_t* ncols;
    int32_t* nnzw;
    uint8_t* route;
    int64_t* wptr;
    int32_t* wcols;
    int32_t* erc;            // per non-zero: (ecol << 4) | row-in-window
    int32_t* mfma_windows;
    int64_t total_ncols;
    int32_t n_mfma, n_csr;
    int64_t nnz_mfma, mfma_ncols;   // non-zeros and distinct columns of the matrix-path windows
    // owned, launch tables
    int32_t* mfma_small;
    hcspmm::WinDesc* mfma_small_desc;
    int32_t* mfma_mid;
    int32_t* mfma_big;
    int32_t n_mfma_small, n_mfma_mid, n_mfma_big;
    hcspmm::WgSlice* mid_slices;     // one per medium window
    hcspmm::WgSlice* big_slices;     // wide windows cut into kSliceCols-column slices
    int32_t n_big_slices;
    int32_t* big_slice_rows;         // per slice and window row: first non-zero inside the slice (sorted rows only)
    hcspmm::MultiRow* tile_multi;    // windows with several slices (row = window id)
    int32_t n_tile_multi;
    int64_t n_tile_slots;
    float* tile_partial;             // lazily sized: n_tile_slots x 16 x d
    int64_t tile_partial_elems;
    // runs of matrix-path windows with merged column lists (the kernel that shares gathered rows through LDS)
    int32_t* ucols;                  // per run: ascending union of its windows' column lists, at RunDesc::up
    int32_t* wslot;                  // per window column (indexed like wcols): its position in the run's union
    hcspmm::RunDesc* runs;
    hcspmm::RunSlice* run_slices;
    hcspmm::RunWin* run_wins;        // kRunWindows records per slice
    hcspmm::MultiRow* run_multi;     // windows of runs cut into several slices (row = window id)
    int32_t n_runs, n_run_slices, n_run_multi;
    int64_t n_run_tile_slots;
    int64_t run_union_cols;          // sum of the runs' union sizes
    int32_t runs_ok;                 // the run tables exist (sorted rows, column count within the bitmap-rank range)
    int32_t rows_sorted;         // 1 when every row's column indices are non-decreasing
    int32_t slice_cols;          // condensed columns per workgroup slice of a wide window (default kSliceCols)
    int32_t mid_row, long_row;   // tier thresholds this plan was built with (defaults kMidRow, kLongRow)
    int32_t fused_mid_row;       // short-tier limit of the fused aggregate-then-update launch (>= mid_row)
    int32_t* short_rows;     // rows of route-0 windows with at most mid_row non-zeros (NULL: walk every row)
    int32_t n_short;
    int32_t* mid_rows;       // rows of route-0 windows with mid_row < non-zeros <= long_row
    int32_t n_mid;
    hcspmm::Segment* segs;
    int32_t n_segs;
    hcspmm::MultiRow* multi;
    int32_t n_multi;
    int64_t n_slots;
    int32_t n_long_rows;
    int32_t condensed_complete;     // 0: wcols / erc are filled for matrix-path windows only (the rest on export)
    int32_t erc_own, wcols_own;     // erc / wcols were allocated on their own (on export), not from the plan's chunks
    void* chunks[64];               // device allocations that hold the plan-owned arrays (several arrays per chunk)
    size_t chunk_bytes[64];
    int32_t n_chunks;
    struct BlockCache* cache;       // device blocks kept between hcspmm_plan_update calls (null until the first one)
    int32_t features_complete;    // ncols / wptr / total_ncols are filled (a scalar-only plan computes them on first request)
    // column panels (n_panels > 1): the scalar path takes the columns panel by panel; scalar_exec: windows that the selector
    // sends to the matrix path run on the scalar path as well, and their condensed structure is built on export only
    int32_t n_panels, scalar_exec;
    int32_t local;                  // neighbouring rows are known to share most of their columns (see build_plan)
    int32_t* panel_split;
    struct { hcspmm::PanelTotals t; int32_t* mid_rows; hcspmm::Segment* segs; hcspmm::MultiRow* multi; } panel[hcspmm::kMaxPanels];
    float* acc_rows;                // n_rows x d sums between panels when the output is not fp32: reserved for 16-bit plans
    int64_t acc_rows_elems;         // (acc_width columns, see reserve_row_sums), lazily sized for the layers otherwise
    int32_t acc_width;
    int32_t n_rest;                 // rows finished through the workspace by the fused update
    int32_t* rest_rows;
    int64_t nnz_long;
    // lazily sized partial-sum buffer for long rows cut into several segments
    float* partial;
    int64_t partial_elems;
    int64_t device_bytes;
    // side streams / events used to run the matrix and scalar paths concurrently
    int32_t side_ok;
    hipStream_t side[2];
    hipEvent_t ev_fork, ev_join[2];
};
