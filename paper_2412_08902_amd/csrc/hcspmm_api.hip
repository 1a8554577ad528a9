// C-ABI entry points: argument checking, plan construction, launch sequencing.
#include "common.hpp"

#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <deque>
#include <mutex>
#include <new>
#include <vector>

// Device blocks kept for reuse instead of going back to the runtime (an allocation and its release cost the
// runtime 20-40 us each, a dozen of them per preparation).  Two uses:
//  * a plan that is updated (hcspmm_plan_update) keeps the scratch of its last update and the arrays of the plan it
//    replaced for the next update; a block that two updates in a row did not use is released; freed with the plan;
//  * one bounded cache per GPU for the whole process serves the preparations of small matrices (blocks of at most
//    16 MiB, 64 MiB in all; what does not fit is released at once).  It lives until the process ends.
struct BlockCache {
    struct Block { void* p; size_t n; int age; };
    std::vector<Block> blocks;
    std::mutex mu;
    size_t max_block = 0, cap = 0, held = 0;      // bounds of the per-GPU cache (0: none)
    // smallest cached block that holds n bytes without wasting more than half of itself (or 1 MiB)
    void* take(size_t n, size_t* got)
    {
        std::lock_guard<std::mutex> g(mu);
        int best = -1;
        for (int i = 0; i < (int)blocks.size(); ++i) {
            const size_t b = blocks[(size_t)i].n;
            if (b < n || b > n + (n / 2 > ((size_t)1 << 20) ? n / 2 : ((size_t)1 << 20))) continue;
            if (best < 0 || b < blocks[(size_t)best].n) best = i;
        }
        if (best < 0) return nullptr;
        void* q = blocks[(size_t)best].p;
        *got = blocks[(size_t)best].n;
        held -= *got;
        blocks.erase(blocks.begin() + best);
        return q;
    }
    void give(void* q, size_t n)
    {
        if (!q) return;
        {
            std::lock_guard<std::mutex> g(mu);
            if (!(max_block && n > max_block) && !(cap && held + n > cap)) {
                blocks.push_back(Block{q, n, 0});
                held += n;
                return;
            }
        }
        (void)hipFree(q);
    }
    void end_of_update()
    {
        std::lock_guard<std::mutex> g(mu);
        for (size_t i = 0; i < blocks.size();) {
            if (++blocks[i].age > 2) { held -= blocks[i].n; (void)hipFree(blocks[i].p); blocks.erase(blocks.begin() + (long)i); }
            else ++i;
        }
    }
    void clear()
    {
        std::lock_guard<std::mutex> g(mu);
        for (Block& b : blocks) (void)hipFree(b.p);
        blocks.clear();
        held = 0;
    }
};

// the process-wide cache of the given GPU (null for a device number beyond the table)
static BlockCache* small_block_cache(int device)
{
    constexpr int kMaxDevices = 64;
    static BlockCache caches[kMaxDevices];
    static std::once_flag once;
    std::call_once(once, [] {
        for (BlockCache& c : caches) { c.max_block = (size_t)16 << 20; c.cap = (size_t)64 << 20; }
    });
    return device >= 0 && device < kMaxDevices ? &caches[device] : nullptr;
}

namespace hcspmm {

static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
}

static int env_int(const char* name)
{
    const char* v = getenv(name);
    return v ? atoi(v) : -1;
}

const Tune& tune()
{
    static const Tune t = {env_int("HCSPMM_TUNE_MID_ROW"), env_int("HCSPMM_TUNE_LONG_ROW"), env_int("HCSPMM_TUNE_SLICE_COLS"),
                           getenv("HCSPMM_TUNE_SERIAL") ? 1 : 0, env_int("HCSPMM_TUNE_XCD_CHUNK"), env_int("HCSPMM_TUNE_RPG"),
                           env_int("HCSPMM_TUNE_TILES_PER_WAVE"),
                           getenv("HCSPMM_TUNE_RUNS") ? 1 : 0, env_int("HCSPMM_TUNE_RUN_SLICE"), env_int("HCSPMM_TUNE_SIDE_NNZ"), env_int("HCSPMM_TUNE_BANDS")};
    return t;
}

// Shipped selector coefficients (w1, w2, b) x 2^20 of  z = w1*ncols + w2*sparsity + b  (Section
// IV-C form; route = matrix path iff z < 0), one row per (precision, dense-width bucket).  Fitted
// on MI355X with the procedure of Section IV-C (synthetic 16-row windows, both deployed kernels
// timed; selector_fit.py) and then checked on community graphs of rising density -- the paper does
// not print its own values.  Read as
//     matrix path  iff  ncols / N0 + sparsity / S0 < 1 :
// N0 bounds the window width, S0 is the sparsity below which the matrix path pays.
//  * d > 64: the matrix path wins or ties from ~1.02 non-zeros per condensed column at every
//    width in the sweep and on the dense power-law graph of the benchmark set (-17 %); wide windows
//    are cut into column slices as far as parallelism needs, so no width limit (w1 = 0) and
//    S0 = 0.936 for large matrices.  On community graphs at d = 128 (blocks of 64, 128-column
//    windows) the scalar path with its XCD-local row order wins at sparsity 0.84 (76 vs 84 us) and
//    loses from 0.72 down (120 vs 96, 143 vs 106, 178 vs 118 us): S0 = 0.83 for smaller matrices.
//  * d <= 64: the sweep (whose windows share no columns with their neighbours) favours the
//    matrix path from ~1.3 non-zeros per column, but on community graphs, where neighbouring rows
//    and windows share columns, the scalar path gets the same reuse out of L1 and the two paths
//    tie within ~10 % up to fully dense blocks; a tie goes to the scalar path (S0 = 0.25: twelve
//    non-zeros per column, i.e. nearly full tiles only).
struct SelectorRow { int32_t dtype; int32_t d_max; int64_t nnz_min; int64_t c[3]; };
static const SelectorRow kSelectorTable[] = {
    // fp32 MFMA
    {HCSPMM_F32, 32, 0, {2048, 4194304, -1048576}},              // N0 = 512,  S0 = 0.25
    {HCSPMM_F32, 64, 0, {171, 4194304, -1048576}},               // N0 = 6144, S0 = 0.25
    // d > 64.  A workgroup-per-window launch has tens of microseconds of fixed latency per
    // workgroup, which only a large matrix amortises: below 16 M non-zeros windows wider than a
    // few hundred columns stay on the scalar path (N0 = 2048), above there is no width limit.
    {HCSPMM_F32, 1 << 30, 16000000, {0, 1120000, -1048576}},     // S0 = 0.936
    {HCSPMM_F32, 1 << 30, 0, {512, 1263344, -1048576}},          // N0 = 2048, S0 = 0.83
    // 16-bit X: the rows of fp32.  On the large dense power-law graph half the gather bytes make the
    // scalar path 2.2x faster than with fp32 X and the matrix path (whose 16-bit stages run three
    // ahead) 2.0x: all-matrix 2.63 ms, all-scalar 2.85 ms, this routing 2.64 ms.  Community graphs
    // at d = 128 favour the matrix path as in fp32 (49/64/91 vs 60/78/116 us), at d = 64 neither.
    {HCSPMM_BF16, 64, 0, {171, 4194304, -1048576}},
    {HCSPMM_BF16, 1 << 30, 16000000, {0, 1120000, -1048576}},    // S0 = 0.936
    {HCSPMM_BF16, 1 << 30, 0, {512, 1120000, -1048576}},
    {HCSPMM_F16, 64, 0, {171, 4194304, -1048576}},
    {HCSPMM_F16, 1 << 30, 16000000, {0, 1120000, -1048576}},
    {HCSPMM_F16, 1 << 30, 0, {512, 1120000, -1048576}},
};

static bool lookup_selector(int32_t dtype, int32_t d_hint, int64_t nnz, int64_t* coef)
{
    if (d_hint <= 0) d_hint = 64;
    for (const SelectorRow& r : kSelectorTable)
        if (r.dtype == dtype && d_hint <= r.d_max && nnz >= r.nnz_min) {
            coef[0] = r.c[0]; coef[1] = r.c[1]; coef[2] = r.c[2];
            return true;
        }
    return false;
}

struct DevAlloc {
    std::vector<void*> ptrs;
    std::vector<size_t> sizes;      // true size of every block in ptrs
    int64_t bytes = 0;
    ::BlockCache* cache = nullptr;  // optional: blocks come from / go back to a plan's cache
    char* arena = nullptr;          // optional: one allocation that get() carves up (scratch of known total size)
    size_t arena_size = 0, arena_used = 0;
    hipError_t raw(void** out, size_t n)
    {
        if (n == 0) n = 256;
        size_t got = n;
        void* q = cache ? cache->take(n, &got) : nullptr;
        if (!q) {
            const hipError_t e = hipMalloc(&q, n);
            if (e != hipSuccess) { *out = nullptr; return e; }
            got = n;
        }
        ptrs.push_back(q);
        sizes.push_back(got);
        *out = q;
        return hipSuccess;
    }
    hipError_t reserve(size_t total)
    {
        void* p = nullptr;
        const hipError_t e = raw(&p, total);
        if (e != hipSuccess) return e;
        arena = static_cast<char*>(p);
        arena_size = total;
        arena_used = 0;
        return hipSuccess;
    }
    size_t chunk_min = 0;           // > 0: arrays are carved out of chunks of at least this size (few device allocations)
    static size_t padded(size_t sz) { return (sz + 255) & ~(size_t)255; }
    template <class T> hipError_t get(T** out, size_t count)
    {
        size_t sz = count * sizeof(T);
        if (sz == 0) sz = sizeof(T) < 16 ? 16 : sizeof(T);
        if (chunk_min && 2 * padded(sz) < chunk_min && !(arena && arena_used + padded(sz) <= arena_size)) {
            const hipError_t e = reserve(chunk_min);            // small arrays share chunks; large ones get their own allocation below
            if (e != hipSuccess) { *out = nullptr; return e; }
        }
        if (!(chunk_min && 2 * padded(sz) >= chunk_min) && arena && arena_used + padded(sz) <= arena_size) {
            *out = reinterpret_cast<T*>(arena + arena_used);
            arena_used += padded(sz);
            bytes += (int64_t)sz;
            return hipSuccess;
        }
        void* q = nullptr;
        const hipError_t e = raw(&q, sz);
        if (e != hipSuccess) { *out = nullptr; return e; }
        bytes += (int64_t)sz;
        *out = static_cast<T*>(q);
        return hipSuccess;
    }
    void free_all()
    {
        for (size_t i = 0; i < ptrs.size(); ++i) {
            if (cache) cache->give(ptrs[i], sizes[i]);
            else (void)hipFree(ptrs[i]);
        }
        ptrs.clear();
        sizes.clear();
        arena = nullptr;
        arena_size = arena_used = 0;
    }
};

#define HC_ALLOC(alloc, ptr, count)                                                                \
    do {                                                                                           \
        if ((alloc).get(&(ptr), (size_t)(count)) != hipSuccess) {                                  \
            (void)hipGetLastError();                                                               \
            set_error("device allocation of %zu elements failed (%s:%d)", (size_t)(count), __FILE__, __LINE__); \
            st = HCSPMM_EALLOC;                                                                    \
            goto fail;                                                                             \
        }                                                                                          \
    } while (0)

#define HC_TRY(call)                                                                               \
    do {                                                                                           \
        hipError_t e_ = (call);                                                                    \
        if (e_ != hipSuccess) {                                                                    \
            set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), __FILE__, __LINE__);  \
            st = HCSPMM_EHIP;                                                                      \
            goto fail;                                                                             \
        }                                                                                          \
    } while (0)

static void free_plan_arrays(hcspmm_plan* p)
{
    // the plan's arrays live in a few chunks; only the lazily sized buffers and arrays completed on export are separate
    BlockCache* to = p->cache ? p->cache : small_block_cache(p->device);
    for (int32_t i = 0; i < p->n_chunks; ++i) {
        if (to) to->give(p->chunks[i], p->chunk_bytes[i]);
        else (void)hipFree(p->chunks[i]);
    }
    p->n_chunks = 0;
    void* owned[] = {p->erc_own ? p->erc : nullptr, p->wcols_own ? p->wcols : nullptr, p->tile_partial, p->partial, p->acc_rows};
    for (void* q : owned)
        if (q) (void)hipFree(q);
}

// Completes what hcspmm_prepare leaves out because no kernel reads it: the window features (ncols,
// wptr, total_ncols) of a scalar-only plan, and -- unless features_only -- wcols / erc of the
// scalar-path windows.  The distinct-column lists are recomputed into scratch memory.  Default
// stream, synchronous.
static hcspmm_status complete_condensed(hcspmm_plan* p, bool features_only)
{
    hcspmm_status st = HCSPMM_OK;
    DevAlloc tmp;
    int32_t *tmp_cols = nullptr, *big_list = nullptr, *cnt = nullptr, *nc_tmp = nullptr, *nz_tmp = nullptr;
    int64_t* scan_tmp = nullptr;
    int32_t h_big = 0;
    const int32_t W = p->W;
    HC_ALLOC(tmp, tmp_cols, p->nnz);
    HC_ALLOC(tmp, big_list, W);
    HC_ALLOC(tmp, cnt, 2);
    HC_ALLOC(tmp, nc_tmp, W);
    HC_ALLOC(tmp, nz_tmp, W);
    HC_ALLOC(tmp, scan_tmp, scan_scratch_elems((int64_t)W + 1));
    HC_TRY(hipMemsetAsync(cnt, 0, 2 * sizeof(int32_t), nullptr));
    if (W > 0) {
        HC_TRY(launch_window_nnz(W, p->n_rows, p->rowptr, nz_tmp, big_list, cnt + 1, nullptr));
        HC_TRY(launch_unique_small(W, p->n_rows, p->rowptr, p->colind, tmp_cols, nc_tmp, nullptr, nullptr));
        HC_TRY(hipMemcpy(&h_big, cnt + 1, sizeof h_big, hipMemcpyDeviceToHost));
        HC_TRY(launch_unique_big(h_big, big_list, p->n_rows, p->n_cols, p->rowptr, p->colind, tmp_cols, nc_tmp, nullptr, nullptr));
    }
    if (!p->features_complete) {
        if (W > 0) HC_TRY(hipMemcpyAsync(p->ncols, nc_tmp, (size_t)W * sizeof(int32_t), hipMemcpyDeviceToDevice, nullptr));
        HC_TRY(exclusive_scan_i32_i64(p->ncols, W, p->wptr, scan_tmp, nullptr));
        HC_TRY(hipMemcpy(&p->total_ncols, p->wptr + W, sizeof(int64_t), hipMemcpyDeviceToHost));
        p->features_complete = 1;
    }
    if (!features_only && !p->condensed_complete) {
        if (!p->erc) {
            if (hipMalloc((void**)&p->erc, (size_t)(p->nnz > 0 ? p->nnz : 1) * sizeof(int32_t)) != hipSuccess) {
                (void)hipGetLastError(); p->erc = nullptr;
                set_error("device allocation failed while completing the condensed structure"); st = HCSPMM_EALLOC; goto fail;
            }
            p->erc_own = 1;
        }
        if (!p->wcols) {
            if (hipMalloc((void**)&p->wcols, (size_t)(p->total_ncols > 0 ? p->total_ncols : 1) * sizeof(int32_t)) != hipSuccess) {
                (void)hipGetLastError(); p->wcols = nullptr;
                set_error("device allocation failed while completing the condensed structure"); st = HCSPMM_EALLOC; goto fail;
            }
            p->wcols_own = 1;
        }
        for (int want = 0; want <= (p->scalar_exec ? 1 : 0) && W > 0; ++want)
            HC_TRY(launch_ecol(W, p->n_rows, p->rowptr, p->colind, tmp_cols, p->ncols, p->wptr, p->wcols, p->erc, cnt, p->route, want,
                               0x7fffffff, nullptr));
        HC_TRY(hipDeviceSynchronize());
        p->condensed_complete = 1;
    }
    HC_TRY(hipDeviceSynchronize());
    tmp.free_all();
    return HCSPMM_OK;
fail:
    (void)hipDeviceSynchronize();
    tmp.free_all();
    return st;
}

// Small device-to-host read-backs of a preparation go through a block of pinned host memory: a copy into
// pageable memory costs the runtime tens of microseconds each.  The totals that every preparation needs are stored there by
// the kernels themselves, and the list of changed windows of an update is read from there, without any copy.
// The blocks are allocated on first use, handed out one per running preparation and kept until the process ends.
class PinnedPage {
public:
    // [0, kReadback): totals written by the kernels; [kReadback, kList): queued read-backs; from kList on: a list the kernels read
    static constexpr size_t kBytes = 65536, kReadback = 1024, kList = 4096;
    PinnedPage()
    {
        std::lock_guard<std::mutex> g(mu());
        for (Slot& sl : pool())
            if (!sl.busy) { sl.busy = true; slot_ = &sl; return; }
        void *q = nullptr, *d = nullptr;
        if (hipHostMalloc(&q, kBytes, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) { (void)hipGetLastError(); return; }
        if (hipHostGetDevicePointer(&d, q, 0) != hipSuccess) { (void)hipGetLastError(); (void)hipHostFree(q); return; }
        pool().push_back(Slot{q, d, true});
        slot_ = &pool().back();
    }
    ~PinnedPage()
    {
        if (!slot_) return;
        std::lock_guard<std::mutex> g(mu());
        slot_->busy = false;
    }
    PinnedPage(const PinnedPage&) = delete;
    PinnedPage& operator=(const PinnedPage&) = delete;
    char* ptr() const { return slot_ ? static_cast<char*>(slot_->p) : nullptr; }
    char* device_ptr() const { return slot_ ? static_cast<char*>(slot_->d) : nullptr; }
private:
    struct Slot { void* p; void* d; bool busy; };
    static std::mutex& mu() { static std::mutex m; return m; }
    static std::deque<Slot>& pool() { static std::deque<Slot> v; return v; }   // (deque: growth keeps the slots in place)
    Slot* slot_ = nullptr;
};

// Read-backs queued on a stream into the pinned page, copied to their host destinations after the stream's next
// synchronisation.  Without a page (or for a block that does not fit) the copy goes straight to its destination.
struct Readback {
    char* page = nullptr;
    size_t used = 0;
    struct Pending { void* dst; size_t off, n; };
    Pending pend[16];
    int n_pend = 0;
    hipError_t add(void* dst, const void* src, size_t n, hipStream_t stream)
    {
        const size_t off = (used + 15) & ~(size_t)15;
        if (!page || n_pend == 16 || off + n > PinnedPage::kList - PinnedPage::kReadback) return hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToHost, stream);
        pend[n_pend++] = Pending{dst, off, n};
        used = off + n;
        return hipMemcpyAsync(page + off, src, n, hipMemcpyDeviceToHost, stream);
    }
    hipError_t sync(hipStream_t stream)
    {
        const hipError_t e = hipStreamSynchronize(stream);
        if (e == hipSuccess)
            for (int i = 0; i < n_pend; ++i) memcpy(pend[i].dst, page + pend[i].off, pend[i].n);
        n_pend = 0;
        used = 0;
        return e;
    }
};

// What an incremental preparation carries over from the previous plan: the distinct-column counts of the windows
// that hold no changed row (device array of the old plan) and the list of windows that do (host, distinct ids).
struct PlanCarry {
    const int32_t* old_ncols; const int32_t* touched; int32_t n_touched;
    // the previous plan's condensed structure (matrix-path windows), when it has one whose rows were all sorted
    const uint8_t* old_route = nullptr; const int64_t* old_wptr = nullptr; const int32_t* old_nnzw = nullptr;
    const int32_t* old_wcols = nullptr; const int32_t* old_erc = nullptr;
};

// Column panels.  On a matrix with many non-zeros per row whose X is far larger than an L2, a row's gathers run over all of
// X and most of them miss (232,965 rows of 492 non-zeros, 128 columns fp32: 36 GB behind L2, at the 6.6 TB/s that this path
// gives: 5.45 ms; the matrix path, which fetches a column once per window, 5.24 ms).  Taking the columns in panels whose
// 128-byte slices about fit an XCD's L2 (3.5 MiB) makes almost every gather a hit, for one more read and write of Y per
// panel and the rows' chains once per panel: 3.5 ms with 9 panels.  A panel should keep some forty non-zeros of a row, and
// panels much larger than an L2 bring little.  Measured against the scalar path in one go: 100,000 rows of 200, 128 columns
// fp32: 759 -> 691 us with 3 panels, 200,000 of 300: 2851 -> 2157 us with 7; but 300,000 of 100, with 5: 1527 -> 1489 us in
// fp32, 752 -> 873 us in bf16 (the sums between panels are fp32), 150,000 of 60: 400 -> 413 us -- i.e. from about 150
// non-zeros per row on, and from 400 for 16-bit rows of 128 bytes (200,000 of 300: 660 -> 695 us).
// The rows have to ascend in their columns, and every window then runs on the scalar path (with panels it is ahead of the
// matrix path on such matrices).
static bool choice_is_ours(const hcspmm_options& o)
{
    return !o.use_custom_selector && o.matrix_kernels == HCSPMM_MATRIX_AUTO && !tune().runs;
}
static int32_t d_or_default(const hcspmm_options& o) { return o.d_hint > 0 ? o.d_hint : 64; }
static int panel_count(const hcspmm_plan* p)
{
    const hcspmm_options& o = p->opt;
    if ((o.route_mode != HCSPMM_ROUTE_HYBRID && o.route_mode != HCSPMM_ROUTE_ALL_CSR) || !choice_is_ours(o) || p->n_rows == 0) return 0;
    const bool f32 = o.mfma_dtype == HCSPMM_F32;
    const int64_t row_bytes = (int64_t)d_or_default(o) * (f32 ? 4 : 2);
    if (row_bytes < kPanelRowBytes) return 0;
    const double degree = (double)p->nnz / p->n_rows;
    if (degree < (!f32 && row_bytes < 2 * kPanelRowBytes ? 400.0 : 150.0)) return 0;
    const double want = (double)p->n_cols * 128.0 / (3.5 * (1 << 20));
    const int n = (int)std::min({want + 0.5, degree / 40.0, (double)kMaxPanels});
    return n >= 2 && 4.0 * n >= want ? n : 0;
}

// Whether windows that the selector sends to the matrix path may run on the scalar path (see scalar_form in
// prepare_kernels.hip for when they do).  The scalar path's column slices live in L2 as long as the graph is not too large:
// 300,000 rows of 60, 128 columns, fp32: 1077 -> 918 us, bf16: 590 -> 457 us; 1 M rows of 20: 1453 -> 1355 us; but 1 M rows
// of 100: 5992 -> 6441 us, 2 M of 40: 5455 -> 5486 us.
static bool scalar_candidate(const hcspmm_plan* p)
{
    // (rows of X off the 128-byte lines cost slices a second line each: 300,000 rows of 60, 144 columns, bf16: 825 -> 1029 us)
    if ((int64_t)p->opt.d_hint * (p->opt.mfma_dtype == HCSPMM_F32 ? 4 : 2) % 128 != 0) return false;
    return p->opt.route_mode == HCSPMM_ROUTE_HYBRID && choice_is_ours(p->opt) && p->n_rows > 0 && p->nnz <= 40000000;
}

// The sample of a preparation (sample_stretch in prepare_kernels.hip).  Where it is small, rows that run side by side share
// most of their columns and X rows are taken whole: column slices gain no hits (p->local).  Communities of 256 to 1,024 nodes
// have 0.05 to 0.14 distinct columns per non-zero in stretches of 16,384 and 0.03 to 0.05 in stretches of 65,536 (131,072 rows
// of 50, 128 columns, fp32, scalar-only plan: 141 -> 111 us, 400,000 of 83: 982 -> 770 us), communities of 4,096 0.10 in the
// long ones (2036 us in panels, 1442 in slices, 1264 whole); communities of 64 next to scattered edges 0.27 in the short
// ones, power-law graphs 0.53 and more (0.4 in the long ones).  A scalar-only plan counts no columns and goes by the short
// sample, taken beside its check of the columns (169,343 rows of 15: 44 -> 50 us); a plan that may take panels has the long one.
constexpr int64_t kSampleNnz = 1 << 20;     // below, a scalar-only preparation is little but its launches

static hcspmm_status build_plan(hcspmm_plan* p, hipStream_t stream, const PlanCarry* carry = nullptr)
{
    hcspmm_status st = HCSPMM_OK;
    DevAlloc tmp;      // scratch, freed on exit
    DevAlloc keep;     // plan-owned (chunks handed to the plan on success), freed on failure only
    PinnedPage pinned;
    Readback rb;
    if (pinned.ptr()) rb.page = pinned.ptr() + PinnedPage::kReadback;
    tmp.cache = keep.cache = p->cache ? p->cache : small_block_cache(p->device);
    const int32_t n_rows = p->n_rows, W = p->W;
    const int64_t nnz = p->nnz;
    keep.chunk_min = (size_t)1 << 20;      // small graphs: all plan arrays in one or two device allocations
    int32_t *err = nullptr, *tmp_cols = nullptr, *touched_dev = nullptr;
    int32_t *sc_n = nullptr, *sc_multi = nullptr, *sc_slots = nullptr;
    int64_t *scan_tmp = nullptr, *pos_a = nullptr, *pos_b = nullptr, *pos_d = nullptr, *totals_dev = nullptr;
    PrepTotals tot, *tot_dev = nullptr;
    unsigned long long* sums = nullptr;
    int32_t h_err = 0;
    int64_t h_tot[16];
    const int32_t n_touched = carry ? carry->n_touched : 0;
    const bool zero_copy = pinned.ptr() && (size_t)n_touched * sizeof(int32_t) <= PinnedPage::kBytes - PinnedPage::kList;
    // upper bounds of the scalar path's row tables (a row in one of them has that many non-zeros), so that they can be
    // filled before the host knows how many entries they get
    const int64_t wide_rows = p->opt.route_mode == HCSPMM_ROUTE_ALL_CSR ? 0 : kH * (nnz / (kMfmaSmallMaxCols + 1));
    const int64_t most_mid = std::min<int64_t>(n_rows, nnz / (p->mid_row + 1)), most_multi = nnz / (kSegLen + 1),
                  most_segs = nnz / (p->long_row + 1) + nnz / kSegLen,
                  most_rest = std::min<int64_t>(n_rows, nnz / (p->fused_mid_row + 1) + wide_rows);
    const int n_panels = panel_count(p);
    Prep pr{};

    {
        // the scratch arrays that every preparation needs: one allocation
        const size_t i32 = sizeof(int32_t);
        const size_t total = DevAlloc::padded(kPrepCtl * i32) + 5 * DevAlloc::padded((size_t)W * i32) +
                             DevAlloc::padded(prep_tile_words(W) * 8) + DevAlloc::padded(sizeof(PrepTotals)) + 16 * 256 +
                             DevAlloc::padded((size_t)n_touched * i32);
        if (tmp.reserve(total) != hipSuccess) {
            (void)hipGetLastError();
            set_error("device allocation of %zu scratch bytes failed", total);
            st = HCSPMM_EALLOC;
            goto fail;
        }
    }
    HC_ALLOC(keep, p->ncols, W);
    HC_ALLOC(keep, p->nnzw, W);
    HC_ALLOC(keep, p->route, W);
    HC_ALLOC(keep, p->wptr, (size_t)W + 1);
    HC_ALLOC(keep, p->mid_rows, most_mid);
    HC_ALLOC(keep, p->segs, most_segs);
    HC_ALLOC(keep, p->multi, most_multi);
    HC_ALLOC(keep, p->rest_rows, most_rest);
    HC_ALLOC(tmp, err, kPrepCtl + 2 * prep_tile_words(W));      // flags, and behind them the sums, which start at zero on some matrices
    sums = reinterpret_cast<unsigned long long*>(err + kPrepCtl);
    if (carry && n_touched > 0) {
        if (zero_copy) {
            memcpy(pinned.ptr() + PinnedPage::kList, carry->touched, (size_t)n_touched * sizeof(int32_t));
            touched_dev = reinterpret_cast<int32_t*>(pinned.device_ptr() + PinnedPage::kList);
        } else {
            HC_ALLOC(tmp, touched_dev, n_touched);
            HC_TRY(hipMemcpyAsync(touched_dev, carry->touched, (size_t)n_touched * sizeof(int32_t), hipMemcpyHostToDevice, stream));
        }
    }
    // A scalar-only plan never reads the condensed structure (the paper has no preprocessing for its
    // scalar path either): its window features stay zero here and are computed when first asked for
    // (hcspmm_plan_info / hcspmm_plan_export), which makes prepare cheap for matrices that keep changing.
    p->features_complete = (p->opt.route_mode == HCSPMM_ROUTE_ALL_CSR && nnz > 0) ? 0 : 1;
    p->rows_sorted = 1;
    pr.n_rows = n_rows; pr.n_cols = p->n_cols; pr.W = W; pr.nnz = nnz;
    pr.rowptr = p->rowptr; pr.colind = p->colind;
    pr.ctl = err;
    HC_ALLOC(tmp, pr.big_list, W);
    HC_ALLOC(tmp, pr.huge_list, W);
    HC_ALLOC(tmp, pr.count_1k, W);
    pr.count_mid = pr.big_list; pr.count_huge = pr.huge_list; pr.n_count_mid = err + 1; pr.n_count_huge = err + 2;
    if (carry) {
        // counts of the untouched windows are the previous plan's; the touched ones are counted (and range-checked) again
        pr.touched = touched_dev;
        pr.old_ncols = carry->old_ncols;
        HC_ALLOC(tmp, pr.count_mid, W);
        HC_ALLOC(tmp, pr.count_huge, W);
        pr.n_count_mid = err + 4; pr.n_count_huge = err + 5;
    }
    pr.features = p->features_complete;
    if (n_panels > 1) pr.panels_from = (int64_t)d_or_default(p->opt) * (p->opt.mfma_dtype == HCSPMM_F32 ? 4 : 2) % 128 == 0 ? 50 : 40;
    pr.sample_len = n_panels > 1 ? kSamplePanels : p->opt.route_mode == HCSPMM_ROUTE_ALL_CSR && nnz >= kSampleNnz ? kSampleSlices : 0;
    if (pr.sample_len > nnz) pr.sample_len = (int32_t)nnz;
    pr.scalar_exec = scalar_candidate(p);
    pr.mode = p->opt.route_mode;
    pr.c0 = p->coef[0]; pr.c1 = p->coef[1]; pr.c2 = p->coef[2];
    pr.mid_row = p->mid_row; pr.long_row = p->long_row; pr.fused_mid_row = p->fused_mid_row;
    pr.ncols = p->ncols; pr.nnzw = p->nnzw; pr.route = p->route; pr.wptr = p->wptr;
    prep_bind_sums(pr, sums);
    pr.mid_rows = p->mid_rows; pr.rest_rows = p->rest_rows; pr.segs = p->segs; pr.multi = p->multi;
    HC_ALLOC(tmp, tot_dev, 1);
    pr.out = pinned.ptr() ? reinterpret_cast<PrepTotals*>(pinned.device_ptr()) : tot_dev;
    HC_TRY(hipMemsetAsync(err, 0, kPrepCtl * sizeof(int32_t) + prep_zeros(pr, n_touched), stream));
    HC_TRY(launch_prep(pr, n_touched, stream));
    if (pinned.ptr()) {
        HC_TRY(hipStreamSynchronize(stream));
        memcpy(&tot, pinned.ptr(), sizeof tot);
    } else {
        HC_TRY(hipMemcpyAsync(&tot, tot_dev, sizeof tot, hipMemcpyDeviceToHost, stream));
        HC_TRY(hipStreamSynchronize(stream));
    }
    if (tot.err & 7) tot.err &= 7;                               // (columns are only asked about where the row offsets are sound)
    if (tot.err) {
        set_error("invalid CSR: %s%s%s%s", (tot.err & 1) ? "rowptr[0] != 0; " : "",
                  (tot.err & 2) ? "rowptr[n_rows] != nnz; " : "", (tot.err & 4) ? "rowptr not non-decreasing; " : "",
                  (tot.err & 8) ? "column index out of range; " : "");
        st = HCSPMM_EBADCSR;
        goto fail;
    }
    p->total_ncols = tot.total_ncols;
    p->n_mfma = tot.n_mfma;
    p->n_csr = W - p->n_mfma;
    p->n_mfma_small = tot.n_mfma_small;
    p->n_mfma_big = tot.n_mfma_big;
    p->n_mfma_mid = tot.n_mfma_mid;
    p->nnz_mfma = tot.nnz_mfma;
    p->mfma_ncols = tot.mfma_cols;
    p->nnz_long = tot.nnz_long;
    p->n_short = tot.n_short;
    p->n_segs = tot.n_segs;
    p->n_multi = tot.n_multi;
    p->n_slots = tot.n_slots;
    p->n_mid = tot.n_mid;
    p->n_rest = tot.n_rest;
    p->n_long_rows = (int32_t)(p->n_segs - p->n_slots + p->n_multi);   // single-segment rows + multi-segment rows
    // condensed structure (column lists, condensed column of every non-zero) of the matrix-path
    // windows; scalar-path windows never read theirs at SpMM time and get it on export only, and a
    // plan without matrix-path windows does not even allocate the arrays
    p->condensed_complete = nnz == 0 ? 1 : 0;
    p->scalar_exec = tot.all_scalar != 0;
    p->n_panels = tot.all_scalar == 2 ? n_panels : 0;
    p->local = sample_share(pr, tot.sample_distinct) < (pr.sample_len > kSampleSlices ? 0.15 : 0.2);
    if (p->n_panels > 1) {
        PanelArgs pa{};
        pa.n_rows = n_rows; pa.n_cols = p->n_cols; pa.n_panels = n_panels; pa.n_tiles = pr.n_tiles;
        pa.mid_row = p->mid_row; pa.long_row = p->long_row; pa.rowptr = p->rowptr; pa.colind = p->colind;
        pa.cap_mid = most_mid; pa.cap_segs = most_segs; pa.cap_multi = most_multi;
        HC_ALLOC(keep, p->panel_split, (size_t)(n_panels - 1) * n_rows);
        HC_ALLOC(keep, pa.mid_rows, (size_t)n_panels * most_mid);
        HC_ALLOC(keep, pa.segs, (size_t)n_panels * most_segs);
        HC_ALLOC(keep, pa.multi, (size_t)n_panels * most_multi);
        HC_ALLOC(tmp, pa.sums, panel_sum_words(n_panels, pa.n_tiles));
        HC_ALLOC(tmp, pa.out, n_panels);
        pa.split = p->panel_split;
        HC_TRY(launch_panels(pa, stream));
        PanelTotals pt[kMaxPanels];
        HC_TRY(rb.add(pt, pa.out, (size_t)n_panels * sizeof(PanelTotals), stream));
        HC_TRY(rb.sync(stream));
        for (int q = 0; q < n_panels; ++q) {
            p->panel[q].t = pt[q];
            p->panel[q].mid_rows = pa.mid_rows + q * pa.cap_mid;
            p->panel[q].segs = pa.segs + q * pa.cap_segs;
            p->panel[q].multi = pa.multi + q * pa.cap_multi;
        }
    }
    // Walking every row and skipping the ones another tier owns is cheaper than an index list while most rows are short
    // scalar-path rows.  Rows of matrix-path windows come in whole windows, i.e. whole workgroups that start only to find
    // nothing to do, and the list pays from a sixteenth of the windows on (walk / list, us, communities + power law, fp32, 128
    // columns: 131,072 + 169,343 rows 225 / 212, 131,072 + 400,000 453 / 447, 65,536 + 169,343 177 / 172, 32,768 + 300,000
    // 167 / 164; bf16 121 / 116).
    p->short_rows = nullptr;
    if ((int64_t)p->n_short * 2 < n_rows || (!p->scalar_exec && (int64_t)p->n_mfma * 16 >= W)) {
        HC_ALLOC(keep, p->short_rows, p->n_short);
        Prep fill = pr;
        fill.mid_rows = fill.rest_rows = nullptr; fill.segs = nullptr; fill.multi = nullptr; fill.out = nullptr;
        fill.short_rows = p->short_rows;
        HC_TRY(launch_prep_fill(fill, stream));
    }
    if (p->n_mfma > 0 && !p->scalar_exec) {
        HC_ALLOC(keep, p->mfma_windows, p->n_mfma);
        HC_ALLOC(keep, p->mfma_small, p->n_mfma_small);
        HC_ALLOC(keep, p->mfma_mid, p->n_mfma_mid);
        HC_ALLOC(keep, p->mfma_big, p->n_mfma_big);
        HC_TRY(launch_prep_windows(pr, p->mfma_windows, p->mfma_small, p->mfma_mid, p->mfma_big, stream));
        HC_ALLOC(keep, p->erc, nnz);
        HC_ALLOC(keep, p->wcols, p->total_ncols);
        HC_ALLOC(tmp, tmp_cols, nnz);
        HC_ALLOC(tmp, scan_tmp, scan_multi_scratch_elems((int64_t)W + 1));
        HC_ALLOC(tmp, pos_a, (size_t)W + 2);
        HC_ALLOC(tmp, pos_b, (size_t)W + 2);
        HC_ALLOC(tmp, pos_d, (size_t)W + 2);
        HC_ALLOC(tmp, totals_dev, 16);
        HC_ALLOC(tmp, sc_n, (size_t)W + 1);
        HC_ALLOC(tmp, sc_multi, (size_t)W + 1);
        HC_ALLOC(tmp, sc_slots, (size_t)W + 1);
        // err[0] is zero here (validation passed): reuse it as the "some row is unsorted" flag.
        // Windows up to kUniqueSmallCap non-zeros: sorted list by the LDS sort, positions by binary search in it.
        // Larger ones: list and positions together from bitmap ranks, unless the matrix is so wide that the
        // bitmap passes would cost more than searching (then the bitmap list + search route serves them too).
        const bool by_rank = p->n_cols <= kRankMaxCols;
        // After a structural change the untouched windows that were and are on the matrix path keep the previous
        // plan's lists and condensed columns (copied to their new offsets); only the others are condensed, through
        // a route array masked down to them.
        const uint8_t* todo_route = p->route;
        if (carry && carry->old_erc && carry->old_wcols) {
            uint8_t *carried = nullptr, *todo = nullptr;
            int64_t* old_start = nullptr;
            HC_ALLOC(tmp, carried, (size_t)W);
            HC_ALLOC(tmp, todo, (size_t)W);
            HC_ALLOC(tmp, old_start, (size_t)W + 1);
            HC_TRY(launch_carry_mask(W, carry->old_route, p->route, n_touched, touched_dev, carried, todo, stream));
            HC_TRY(exclusive_scan_i32_i64(carry->old_nnzw, W, old_start, scan_tmp, stream));
            HC_TRY(launch_carry_copy(W, n_rows, carried, carry->old_wptr, p->wptr, carry->old_wcols, p->wcols, old_start,
                                     p->rowptr, carry->old_erc, p->erc, stream));
            todo_route = todo;
        }
        HC_TRY(launch_unique_small(W, n_rows, p->rowptr, p->colind, tmp_cols, p->ncols, todo_route, stream));
        if (by_rank) {
            HC_TRY(launch_condense_rank(tot.n_big_list, pr.big_list, n_rows, p->rowptr, p->colind, todo_route, p->wptr, p->wcols,
                                        p->erc, err, stream));
            HC_TRY(launch_condense_rank(tot.n_huge_list, pr.huge_list, n_rows, p->rowptr, p->colind, todo_route, p->wptr, p->wcols,
                                        p->erc, err, stream));
        } else {
            HC_TRY(launch_unique_big(tot.n_big_list, pr.big_list, n_rows, p->n_cols, p->rowptr, p->colind, tmp_cols, p->ncols,
                                     todo_route, stream));
            HC_TRY(launch_unique_big(tot.n_huge_list, pr.huge_list, n_rows, p->n_cols, p->rowptr, p->colind, tmp_cols, p->ncols,
                                     todo_route, stream));
        }
        HC_TRY(launch_ecol(W, n_rows, p->rowptr, p->colind, tmp_cols, p->ncols, p->wptr, p->wcols, p->erc, err, todo_route, 1,
                           by_rank ? kUniqueSmallCap : 0x7fffffff, stream));
        HC_TRY(rb.add(&h_err, err, sizeof h_err, stream));
        HC_TRY(rb.sync(stream));
        p->rows_sorted = h_err ? 0 : 1;
    }
    // Runs of matrix-path windows (kRunWindows consecutive list entries each): merged column lists and slots on the
    // device, the slice layout on the host from the union sizes (a few bytes per run cross the bus).
    p->runs_ok = 0;
    if (p->n_mfma > 0 && !p->scalar_exec && p->rows_sorted && p->n_cols <= kRankMaxCols && (p->opt.matrix_kernels == HCSPMM_MATRIX_RUNS || tune().runs)) {
        const int32_t n_runs = (p->n_mfma + kRunWindows - 1) / kRunWindows;
        HC_ALLOC(keep, p->ucols, p->total_ncols);
        HC_ALLOC(keep, p->wslot, p->total_ncols);
        HC_ALLOC(keep, p->runs, n_runs);
        HC_TRY(hipMemsetAsync(p->wslot, 0xff, (size_t)p->total_ncols * sizeof(int32_t), stream));   // -1 where no run owns the column
        HC_TRY(launch_run_union(n_runs, p->mfma_windows, p->n_mfma, p->ncols, p->wptr, p->wcols, p->ucols, p->wslot, p->runs,
                                stream));
        std::vector<RunDesc> h_runs((size_t)n_runs);
        std::vector<int32_t> h_list((size_t)p->n_mfma);
        HC_TRY(rb.add(h_runs.data(), p->runs, (size_t)n_runs * sizeof(RunDesc), stream));
        HC_TRY(rb.add(h_list.data(), p->mfma_windows, (size_t)p->n_mfma * sizeof(int32_t), stream));
        HC_TRY(rb.sync(stream));
        int64_t u_total = 0;
        for (const RunDesc& r : h_runs) u_total += r.nu;
        int64_t slice_u = (u_total / kRunTargetSlices + 63) / 64 * 64;
        if (slice_u < kRunMinSlice) slice_u = kRunMinSlice;
        if (tune().run_slice >= 64) slice_u = tune().run_slice / 64 * 64;
        std::vector<RunSlice> h_slices;
        std::vector<MultiRow> h_multi;
        int64_t slots = 0;
        for (int32_t r = 0; r < n_runs; ++r) {
            RunDesc& rd = h_runs[(size_t)r];
            const int32_t ns = (int32_t)((rd.nu + slice_u - 1) / slice_u);
            rd.n_slices = ns < 1 ? 1 : ns;
            rd.slot0 = 0;
            if (rd.n_slices > 1) {
                if (slots + (int64_t)rd.nw * rd.n_slices >= ((int64_t)1 << 27)) { set_error("too many partial tiles"); st = HCSPMM_EUNSUPPORTED; goto fail; }
                rd.slot0 = (int32_t)slots;
                for (int32_t i = 0; i < rd.nw; ++i)
                    h_multi.push_back(MultiRow{h_list[(size_t)rd.first + i], rd.slot0 + i * rd.n_slices, rd.n_slices, 0});
                slots += (int64_t)rd.nw * rd.n_slices;
            }
            for (int32_t q = 0; q < rd.n_slices; ++q) {
                const int64_t b = (int64_t)q * slice_u;
                h_slices.push_back(RunSlice{rd.up, r, (int32_t)b, (int32_t)(b + slice_u < rd.nu ? b + slice_u : rd.nu), q, rd.nw,
                                            rd.n_slices, rd.slot0, {0, 0, 0}});
            }
        }
        p->n_runs = n_runs;
        p->n_run_slices = (int32_t)h_slices.size();
        p->n_run_multi = (int32_t)h_multi.size();
        p->n_run_tile_slots = slots;
        p->run_union_cols = u_total;
        HC_ALLOC(keep, p->run_slices, h_slices.size());
        HC_ALLOC(keep, p->run_multi, h_multi.size());
        HC_TRY(hipMemcpyAsync(p->runs, h_runs.data(), (size_t)n_runs * sizeof(RunDesc), hipMemcpyHostToDevice, stream));
        HC_TRY(hipMemcpyAsync(p->run_slices, h_slices.data(), h_slices.size() * sizeof(RunSlice), hipMemcpyHostToDevice, stream));
        if (!h_multi.empty())
            HC_TRY(hipMemcpyAsync(p->run_multi, h_multi.data(), h_multi.size() * sizeof(MultiRow), hipMemcpyHostToDevice, stream));
        HC_ALLOC(keep, p->run_wins, h_slices.size() * kRunWindows);
        HC_TRY(launch_run_wins(p->n_run_slices, p->run_slices, p->runs, p->mfma_windows, p->ncols, p->wptr, n_rows, p->rowptr,
                               p->run_wins, stream));
        HC_TRY(rb.sync(stream));                    // the host vectors go out of scope
        p->runs_ok = 1;
    }
    // workgroup slices: one per medium window, slice_cols condensed columns each for wide windows
    if (p->n_mfma > 0 && !p->scalar_exec) {
        ScanMulti m{};
        m.k = 3;
        m.in[0] = sc_n;     m.out[0] = pos_a;
        m.in[1] = sc_multi; m.out[1] = pos_b;
        m.in[2] = sc_slots; m.out[2] = pos_d;
        HC_ALLOC(keep, p->mid_slices, p->n_mfma_mid);
        if (p->n_mfma_mid > 0) {
            HC_TRY(launch_slice_count(p->n_mfma_mid, p->mfma_mid, p->ncols, 0x40000000, sc_n, sc_multi, sc_slots, stream));
            HC_TRY(exclusive_scan_multi(m, p->n_mfma_mid, nullptr, scan_tmp, stream));
            HC_TRY(launch_slice_fill(p->n_mfma_mid, p->mfma_mid, p->ncols, 0x40000000, pos_a, pos_b, pos_d, p->mid_slices,
                                     nullptr, stream));
        }
        // Wide windows are cut into slices only as far as parallelism needs it (a slice loses the
        // alignment of concurrently running windows on the same hot low-numbered columns): aim
        // at ~4 workgroups per CU over the summed width of the wide windows.
        if (tune().slice_cols < 0 && p->n_mfma_big > 0) {
            int64_t want = tot.wide_cols / 1024;
            if (want < kKcBig) want = kKcBig;
            if (want > (1 << 27)) want = 1 << 27;
            p->slice_cols = (int32_t)((want + kKcBig - 1) / kKcBig * kKcBig);
        }
        h_tot[0] = h_tot[1] = h_tot[2] = 0;
        if (p->n_mfma_big > 0) {
            HC_TRY(launch_slice_count(p->n_mfma_big, p->mfma_big, p->ncols, p->slice_cols, sc_n, sc_multi, sc_slots, stream));
            HC_TRY(exclusive_scan_multi(m, p->n_mfma_big, totals_dev, scan_tmp, stream));
            HC_TRY(rb.add(h_tot, totals_dev, 3 * sizeof(int64_t), stream));
            HC_TRY(rb.sync(stream));
        }
        p->n_big_slices = (int32_t)h_tot[0];
        p->n_tile_multi = (int32_t)h_tot[1];
        p->n_tile_slots = h_tot[2];
        if (tune().bands > 0 && p->n_mfma_big > 0) {
            // Measurement aid (HCSPMM_TUNE_BANDS): wide windows are cut at the same global column boundaries and the
            // slices ordered band by band, so that all windows walk one band's X rows at about the same time.  Built on
            // the host from a copy of the column lists: slow, and only for the experiment that profiles/ reports.
            const int32_t Bc = tune().bands;
            std::vector<int32_t> h_list((size_t)p->n_mfma_big), h_nc((size_t)W), h_wc((size_t)p->total_ncols);
            std::vector<int64_t> h_wp((size_t)W + 1);
            HC_TRY(hipMemcpyAsync(h_list.data(), p->mfma_big, h_list.size() * 4, hipMemcpyDeviceToHost, stream));
            HC_TRY(hipMemcpyAsync(h_nc.data(), p->ncols, h_nc.size() * 4, hipMemcpyDeviceToHost, stream));
            HC_TRY(hipMemcpyAsync(h_wp.data(), p->wptr, h_wp.size() * 8, hipMemcpyDeviceToHost, stream));
            HC_TRY(hipMemcpyAsync(h_wc.data(), p->wcols, h_wc.size() * 4, hipMemcpyDeviceToHost, stream));
            HC_TRY(hipStreamSynchronize(stream));
            // HCSPMM_TUNE_BANDS_HOT=k: only the first k bands are cut; all columns behind them form one last band
            const int32_t hot = getenv("HCSPMM_TUNE_BANDS_HOT") ? atoi(getenv("HCSPMM_TUNE_BANDS_HOT")) : 0x7fffffff;
            const int32_t n_bands = std::min((p->n_cols + Bc - 1) / Bc, hot < 0x7fffffff ? hot + 1 : 0x7fffffff);
            std::vector<std::vector<WgSlice>> per_band((size_t)n_bands);
            std::vector<MultiRow> h_multi;
            int64_t slots = 0;
            for (int32_t w : h_list) {
                const int32_t* c0 = h_wc.data() + h_wp[(size_t)w];
                const int32_t nc = h_nc[(size_t)w];
                int32_t n_here = 0;
                const int64_t first = slots;
                int32_t kb = 0;
                while (kb < nc) {
                    const int32_t b = std::min(c0[kb] / Bc, n_bands - 1);
                    const int32_t ke = b == n_bands - 1 ? nc : (int32_t)(std::lower_bound(c0 + kb, c0 + nc, (b + 1) * Bc) - c0);
                    per_band[(size_t)b].push_back(WgSlice{w, kb, ke, (int32_t)(first + n_here)});
                    ++n_here;
                    kb = ke;
                }
                slots += n_here;
                h_multi.push_back(MultiRow{w, (int32_t)first, n_here, 0});
            }
            std::vector<WgSlice> h_sl;
            for (auto& v : per_band) h_sl.insert(h_sl.end(), v.begin(), v.end());
            p->n_big_slices = (int32_t)h_sl.size();
            p->n_tile_multi = (int32_t)h_multi.size();
            p->n_tile_slots = slots;
            HC_ALLOC(keep, p->big_slices, p->n_big_slices);
            HC_ALLOC(keep, p->tile_multi, p->n_tile_multi);
            HC_TRY(hipMemcpy(p->big_slices, h_sl.data(), h_sl.size() * sizeof(WgSlice), hipMemcpyHostToDevice));
            HC_TRY(hipMemcpy(p->tile_multi, h_multi.data(), h_multi.size() * sizeof(MultiRow), hipMemcpyHostToDevice));
        } else {
        HC_ALLOC(keep, p->big_slices, p->n_big_slices);
        HC_ALLOC(keep, p->tile_multi, p->n_tile_multi);
        if (p->n_mfma_big > 0)
            HC_TRY(launch_slice_fill(p->n_mfma_big, p->mfma_big, p->ncols, p->slice_cols, pos_a, pos_b, pos_d, p->big_slices,
                                     p->tile_multi, stream));
        }
        if (p->rows_sorted && p->n_big_slices > 0) {
            HC_ALLOC(keep, p->big_slice_rows, (size_t)p->n_big_slices * kH);
            HC_TRY(launch_slice_rows(p->n_big_slices, p->big_slices, n_rows, p->rowptr, p->erc, p->big_slice_rows,
                                     stream));
        }
    }
    if (p->n_mfma_small > 0 && !p->scalar_exec) {
        HC_ALLOC(keep, p->mfma_small_desc, p->n_mfma_small);
        HC_TRY(launch_build_desc(p->n_mfma_small, p->mfma_small, n_rows, p->rowptr, p->ncols, p->wptr, p->mfma_small_desc,
                                 stream));
    }
    if (p->n_mfma > 0 || p->short_rows) HC_TRY(rb.sync(stream));
    p->device_bytes = keep.bytes;
    if (keep.ptrs.size() > sizeof p->chunks / sizeof p->chunks[0]) {
        set_error("internal: too many plan chunks");
        st = HCSPMM_EALLOC;
        goto fail;
    }
    p->n_chunks = (int32_t)keep.ptrs.size();
    for (size_t i = 0; i < keep.ptrs.size(); ++i) { p->chunks[i] = keep.ptrs[i]; p->chunk_bytes[i] = keep.sizes[i]; }
    tmp.free_all();
    return HCSPMM_OK;

fail:
    (void)hipStreamSynchronize(stream);
    tmp.free_all();
    keep.free_all();
    return st;
}

// partial tiles a call may need: the slices of wide windows, or of wide runs when the run kernel serves the matrix path
static int64_t tile_slots(const hcspmm_plan* p) { return p->n_tile_slots > p->n_run_tile_slots ? p->n_tile_slots : p->n_run_tile_slots; }

// partial rows a call may need: long rows cut into segments, or the panels' (one panel runs at a time)
static int64_t row_slots(const hcspmm_plan* p)
{
    int64_t n = p->n_slots;
    for (int q = 0; q < p->n_panels; ++q) n = std::max(n, p->panel[q].t.n_slots);
    return n;
}

// Scratch of one SpMM call: partial rows of long rows cut into several segments, then partial tiles of
// wide windows cut into several slices (each part padded to 256 bytes).
static size_t spmm_scratch_bytes(const hcspmm_plan* p, int32_t d, size_t* tile_off)
{
    const size_t part = ((size_t)row_slots(p) * (size_t)d * sizeof(float) + 255) & ~(size_t)255;
    const size_t tiles = ((size_t)tile_slots(p) * kH * (size_t)d * sizeof(float) + 255) & ~(size_t)255;
    if (tile_off) *tile_off = part;
    return part + tiles;
}

// Plans for 16-bit features with column panels hold the panels' fp32 sums of a 16-bit output from the start, for the width
// they were made for: hcspmm_spmm_noalloc allocates nothing and gives the bits of hcspmm_spmm, so what the two do must not
// depend on earlier calls.  (232,965 rows of 492, bf16 to bf16, 256 columns: 5483 us in one pass over all columns, 4675 us on
// the matrix path, 4139 us in panels; 128 columns: 2532, 2627, 2141 us.)
static hcspmm_status reserve_row_sums(hcspmm_plan* p, int64_t have)
{
    p->acc_width = 0;
    if (p->n_panels < 2 || p->opt.mfma_dtype == HCSPMM_F32) return HCSPMM_OK;
    p->acc_width = d_or_default(p->opt);
    const int64_t want = (int64_t)p->n_rows * p->acc_width;
    if (have >= want) return HCSPMM_OK;
    if (hipMalloc((void**)&p->acc_rows, (size_t)want * sizeof(float)) != hipSuccess) {
        (void)hipGetLastError();
        p->acc_rows = nullptr;
        set_error("allocation of %lld floats for row sums between column panels failed", (long long)want);
        return HCSPMM_EALLOC;
    }
    p->acc_rows_elems = want;
    return HCSPMM_OK;
}

// Room in the plan's own scratch for calls of width d: partial rows of long rows cut into several segments, partial tiles of
// wide windows.  Growing it waits for the calls that use it.
static hcspmm_status reserve_scratch(hcspmm_plan* p, int32_t d, hipStream_t stream)
{
    const int64_t rows = row_slots(p) * (int64_t)d;
    if (p->partial_elems < rows) {
        if (p->partial) { HC_HIP(hipStreamSynchronize(stream)); (void)hipFree(p->partial); p->partial = nullptr; }
        if (hipMalloc((void**)&p->partial, (size_t)rows * sizeof(float)) != hipSuccess) {
            (void)hipGetLastError();
            p->partial = nullptr;
            p->partial_elems = 0;
            set_error("allocation of %lld floats for long-row partial sums failed", (long long)rows);
            return HCSPMM_EALLOC;
        }
        p->partial_elems = rows;
    }
    const int64_t tiles = tile_slots(p) * kH * (int64_t)d;
    if (p->tile_partial_elems < tiles) {
        if (p->tile_partial) { HC_HIP(hipStreamSynchronize(stream)); (void)hipFree(p->tile_partial); p->tile_partial = nullptr; }
        if (hipMalloc((void**)&p->tile_partial, (size_t)tiles * sizeof(float)) != hipSuccess) {
            (void)hipGetLastError();
            p->tile_partial = nullptr;
            p->tile_partial_elems = 0;
            set_error("allocation of %lld floats for wide-window partial tiles failed", (long long)tiles);
            return HCSPMM_EALLOC;
        }
        p->tile_partial_elems = tiles;
    }
    return HCSPMM_OK;
}

// Whether a call keeps its rows' sums between column panels in the plan (fp32 results keep them in Y itself).
static bool panel_sums_needed(const hcspmm_plan* p, const SpmmArgs& a)
{
    return p->n_panels > 1 && a.y_dtype != HCSPMM_F32 && csr_panels_usable(a);
}

// Room for those sums.  The ones at hand are given up only for larger ones: calls that must not allocate count on them.
static hcspmm_status reserve_panel_sums(hcspmm_plan* p, int32_t d, hipStream_t stream)
{
    const int64_t want = (int64_t)p->n_rows * d;
    if (p->acc_rows_elems >= want) return HCSPMM_OK;
    float* larger = nullptr;
    if (hipMalloc((void**)&larger, (size_t)want * sizeof(float)) != hipSuccess) {
        (void)hipGetLastError();
        set_error("allocation of %lld floats for row sums between column panels failed", (long long)want);
        return HCSPMM_EALLOC;
    }
    if (p->acc_rows) { HC_HIP(hipStreamSynchronize(stream)); (void)hipFree(p->acc_rows); }
    p->acc_rows = larger;
    p->acc_rows_elems = want;
    return HCSPMM_OK;
}

// (the windows' distinct columns against their non-zeros say how much the rows of a window share; a scalar-only plan does
// not count them and goes by its sample)
static CsrHints csr_hints(const hcspmm_plan* p, bool beside)
{
    const int64_t nnz_scalar = p->nnz - (p->scalar_exec ? 0 : p->nnz_mfma), n_scalar = p->scalar_exec ? p->W : p->n_csr;
    const int64_t cols_scalar = p->total_ncols - (p->scalar_exec ? 0 : p->mfma_ncols);
    const bool scattered = !p->local && (p->opt.route_mode == HCSPMM_ROUTE_ALL_CSR || 10 * cols_scalar > 6 * nnz_scalar);
    return CsrHints{nnz_scalar, n_scalar * kH, scattered, p->long_row, beside, p->nnz};
}

static hcspmm_status run_spmm(const hcspmm_plan* plan, const SpmmArgs& a, hipStream_t stream,
                              hipEvent_t* ev = nullptr /* 5 events when timing stages */,
                              const UpdateArgs* upd = nullptr /* fuse the update stage where a tile stays on chip */,
                              bool windows_only = false /* ... in the wave-per-window matrix kernel only */,
                              char* scratch_mem = nullptr /* device, spmm_scratch_bytes(): used instead of the plan's own lazily sized buffers */,
                              bool acc_rows = false /* column panels may keep fp32 sums of a 16-bit output in a buffer of the plan */)
{
    hcspmm_plan* p = const_cast<hcspmm_plan*>(plan);
    if (a.x_mask && p->n_mfma > 0 && !p->scalar_exec) HC_HIP(hipErrorInvalidValue);      // (the matrix path looks at no mask; launch_csr refuses the other cases)
    if (!scratch_mem) {
        const hcspmm_status st = reserve_scratch(p, a.d, stream);
        if (st != HCSPMM_OK) return st;
    }
    float* partial = p->partial;
    float* tile_partial = p->tile_partial;
    if (scratch_mem) {
        size_t tile_off = 0;
        (void)spmm_scratch_bytes(p, a.d, &tile_off);
        partial = reinterpret_cast<float*>(scratch_mem);
        tile_partial = reinterpret_cast<float*>(scratch_mem + tile_off);
    }
    // Column panels: the same kernel once per panel, each adding to what the previous ones left (in Y itself when it is fp32,
    // in fp32 sums of the plan otherwise).
    if (p->n_panels > 1 && !upd && csr_panels_usable(a) && (a.y_dtype == HCSPMM_F32 || acc_rows)) {
        float* sums = a.Y;
        int64_t ld_sums = a.ldy;
        if (a.y_dtype != HCSPMM_F32) {
            const hcspmm_status st = reserve_panel_sums(p, a.d, stream);
            if (st != HCSPMM_OK) return st;
            sums = p->acc_rows;
            ld_sums = a.d;
        }
        if (ev) for (int i = 0; i < 3; ++i) HC_HIP(hipEventRecord(ev[i], stream));
        for (int q = 0; q < p->n_panels; ++q) {
            const PanelTotals& t = p->panel[q].t;
            SpmmArgs b = a;
            const bool final_panel = q == p->n_panels - 1;
            if (q > 0) { b.rowptr = p->panel_split + (int64_t)(q - 1) * p->n_rows; b.acc = sums; b.ldacc = ld_sums; }
            b.rowend = final_panel ? p->rowptr + 1 : p->panel_split + (int64_t)q * p->n_rows;
            if (!final_panel) { b.Y = sums; b.ldy = ld_sums; b.y_dtype = HCSPMM_F32; b.relu = 0; }
            const CsrHints hints{t.nnz, p->n_rows, true, p->long_row, false, p->nnz};
            HC_HIP(launch_csr(b, t.n_segs, p->panel[q].segs, partial, t.n_mid, p->panel[q].mid_rows, p->n_rows, nullptr, nullptr, p->mid_row,
                              hints, stream));
            HC_HIP(launch_reduce_partials(b, t.n_multi, p->panel[q].multi, partial, stream));
        }
        if (ev) { HC_HIP(hipEventRecord(ev[3], stream)); HC_HIP(hipEventRecord(ev[4], stream)); }
        return HCSPMM_OK;
    }
    const bool use_runs = p->runs_ok && !upd && mfma_run_shape_supported(a);
    const bool has_wg = use_runs ? p->n_run_slices > 0 : !p->scalar_exec && (p->n_big_slices > 0 || p->n_mfma_mid > 0);
    const bool has_small = !use_runs && !p->scalar_exec && p->n_mfma_small > 0;
    const bool has_csr = p->n_segs > 0 || p->n_mid > 0 || p->n_short > 0;
    // The paths own disjoint rows of Y.  When more than one has work (and the stages are not being
    // timed one by one) they run side by side: the matrix-path kernels on the plan's two side
    // streams, forked from and joined back to the caller's stream with events.
    const bool side = !ev && p->side_ok && (int)has_wg + (int)has_small + (int)has_csr > 1;
    hipStream_t s_wg = stream, s_small = stream;
    if (side) {
        HC_HIP(hipEventRecord(p->ev_fork, stream));
        if (has_wg && has_csr) { s_wg = p->side[0]; HC_HIP(hipStreamWaitEvent(s_wg, p->ev_fork, 0)); }
        if (has_small && (has_csr || has_wg)) { s_small = p->side[1]; HC_HIP(hipStreamWaitEvent(s_small, p->ev_fork, 0)); }
    }
    if (ev) HC_HIP(hipEventRecord(ev[0], stream));
    if (use_runs) {
        // every matrix-path window through the run kernel: neighbouring windows share their gathered rows in LDS
        HC_HIP(launch_mfma_run(a, p->n_run_slices, p->run_slices, p->run_wins, p->ucols, p->wslot, p->erc, tile_partial, s_wg));
        HC_HIP(launch_reduce_tiles(a, p->n_run_multi, p->run_multi, tile_partial, s_wg));
        if (ev) { HC_HIP(hipEventRecord(ev[1], stream)); HC_HIP(hipEventRecord(ev[2], stream)); }
    } else if (p->scalar_exec) {
        if (ev) { HC_HIP(hipEventRecord(ev[1], stream)); HC_HIP(hipEventRecord(ev[2], stream)); }
    } else {
        HC_HIP(launch_mfma_wg(a, p->n_big_slices, p->big_slices, p->ncols, p->wptr, p->wcols, p->erc, p->rows_sorted,
                              p->big_slice_rows, tile_partial, tune().bands <= 0 || getenv("HCSPMM_TUNE_BANDS_WIDE"), s_wg));
        HC_HIP(launch_reduce_tiles(a, p->n_tile_multi, p->tile_multi, tile_partial, s_wg));
        HC_HIP(launch_mfma_wg(a, p->n_mfma_mid, p->mid_slices, p->ncols, p->wptr, p->wcols, p->erc, p->rows_sorted,
                              nullptr, tile_partial, false, s_wg));
        if (ev) HC_HIP(hipEventRecord(ev[1], stream));
        HC_HIP(launch_mfma_small(a, p->n_mfma_small, p->mfma_small_desc, p->wcols, p->erc, s_small, upd));
        if (ev) HC_HIP(hipEventRecord(ev[2], stream));
    }
    const int64_t n_scalar = p->scalar_exec ? p->W : p->n_csr;
    const CsrHints hints = csr_hints(p, side && has_csr);
    const uint8_t* route = p->scalar_exec || p->n_mfma == 0 ? nullptr : p->route;
    if (upd && !windows_only)        // the fused launch walks every row: its tile tier also takes the shorter mid rows
        HC_HIP(launch_csr(a, p->n_segs, p->segs, partial, p->n_mid, p->mid_rows, n_scalar > 0 ? p->n_rows : 0, nullptr,
                          route, p->fused_mid_row, hints, stream, upd));
    else
        HC_HIP(launch_csr(a, p->n_segs, p->segs, partial, p->n_mid, p->mid_rows,
                          p->short_rows ? p->n_short : (p->n_short > 0 ? p->n_rows : 0), p->short_rows, route,
                          p->mid_row, hints, stream));
    if (ev) HC_HIP(hipEventRecord(ev[3], stream));
    HC_HIP(launch_reduce_partials(a, p->n_multi, p->multi, partial, stream));
    if (ev) HC_HIP(hipEventRecord(ev[4], stream));
    if (s_wg != stream) {
        HC_HIP(hipEventRecord(p->ev_join[0], s_wg));
        HC_HIP(hipStreamWaitEvent(stream, p->ev_join[0], 0));
    }
    // rows whose aggregation went to memory: all but the fused windows' rows, or long and mid rows and wide matrix-path windows
    if (windows_only)
        HC_HIP(launch_gemm_f32_out(p->n_rows, a.d, upd->d_out, a.Y, a.ldy, upd->W, upd->ldw, upd->Y, upd->ldy, upd->y_dtype, upd->relu,
                                   stream, p->route, p->ncols));
    if (s_small != stream) {
        HC_HIP(hipEventRecord(p->ev_join[1], s_small));
        HC_HIP(hipStreamWaitEvent(stream, p->ev_join[1], 0));
    }
    if (upd && !windows_only) HC_HIP(launch_update_rest(a, p->n_rest, p->rest_rows, *upd, stream));
    return HCSPMM_OK;
}

}  // namespace hcspmm

using namespace hcspmm;

// ---- scratch of the entry point that allocates nothing ------------------------------------------
// One array per GPU, part of the library's device image: it exists from the moment the library is loaded
// on a device until the process ends.  `scratch` itself is only the host-side handle of the symbol; the
// array's device address is looked up once per device and kept in g_scratch_ptr.
constexpr size_t kStaticScratchBytes = HCSPMM_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static char* g_scratch_ptr[kMaxDevices] = {};

// device address of the current GPU's copy of the array; the current device must be the plan's
static hcspmm_status static_scratch_ptr(const hcspmm_plan* plan, char** out)
{
    int dev = -1;
    HC_HIP(hipGetDevice(&dev));
    if (dev != plan->device) { set_error("the current device (%d) is not the plan's (%d)", dev, plan->device); return HCSPMM_EINVAL; }
    if (dev < 0 || dev >= kMaxDevices) { set_error("device index %d is beyond the %d devices supported", dev, kMaxDevices); return HCSPMM_EUNSUPPORTED; }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        HC_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) { set_error("hipGetSymbolAddress returned no address for the static scratch array"); return HCSPMM_EHIP; }
        g_scratch_ptr[dev] = static_cast<char*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return HCSPMM_OK;
}

// everything of a plan that does not depend on the matrix's entries
static hcspmm_status init_plan_header(hcspmm_plan* p, int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t* d_rowptr,
                                      const int32_t* d_colind, const float* d_vals, const hcspmm_options& o)
{
    memset(p, 0, sizeof *p);
    p->H = kH; p->n_rows = n_rows; p->n_cols = n_cols; p->nnz = nnz;
    p->W = (int32_t)(((int64_t)n_rows + kH - 1) / kH);
    p->rowptr = d_rowptr; p->colind = d_colind; p->vals = d_vals;
    p->opt = o;
    p->mid_row = n_rows <= kMidRowFewRows ? kMidRowSmall : kMidRow;
    p->long_row = n_rows >= kLongRowFewRows && nnz < kLongRowDegree * n_rows ? kLongRowSparse : kLongRow;
    // tuning knobs for experiments (not part of the ABI): override the row-tier thresholds
    if (tune().mid_row >= 1) p->mid_row = tune().mid_row;
    if (tune().long_row >= p->mid_row) p->long_row = tune().long_row;
    if (p->long_row < p->mid_row) p->long_row = p->mid_row;
    p->fused_mid_row = kFusedMidRow < p->mid_row ? p->mid_row : (kFusedMidRow > p->long_row ? p->long_row : kFusedMidRow);
    p->slice_cols = kSliceCols;
    if (tune().slice_cols >= kKcBig) p->slice_cols = tune().slice_cols / kKcBig * kKcBig;
    if (o.use_custom_selector) {
        for (int i = 0; i < 3; ++i) {
            if (o.sel_coef[i] <= -((int64_t)1 << 40) || o.sel_coef[i] >= ((int64_t)1 << 40)) {
                set_error("selector coefficients must be below 2^40 in magnitude");
                return HCSPMM_EINVAL;
            }
            p->coef[i] = o.sel_coef[i];
        }
    } else {
        lookup_selector(o.mfma_dtype, o.d_hint, nnz, p->coef);
    }
    if (hipGetDevice(&p->device) != hipSuccess) { (void)hipGetLastError(); set_error("hipGetDevice failed"); return HCSPMM_EHIP; }
    // set-up of hcspmm_spmm_noalloc: this device's address of the static scratch array, looked up once per device
    char* unused = nullptr;
    return static_scratch_ptr(p, &unused);
}

// side streams (default priority) and events for running the paths side by side; optional
// (the fork/join costs ~20 us of launch latency, so only matrices with milliseconds of work use them)
constexpr int64_t kSideStreamNnz = 16000000;
static void setup_side_streams(hcspmm_plan* p)
{
    if (p->side_ok || p->side[0]) return;
    p->side_ok = 0;
    if (p->n_mfma > 0 && p->n_mfma < p->W && !p->scalar_exec && p->nnz >= (tune().side_nnz >= 0 ? tune().side_nnz : kSideStreamNnz) && !tune().serial) {
        bool ok = hipStreamCreateWithFlags(&p->side[0], hipStreamNonBlocking) == hipSuccess;
        ok = ok && hipStreamCreateWithFlags(&p->side[1], hipStreamNonBlocking) == hipSuccess;
        ok = ok && hipEventCreateWithFlags(&p->ev_fork, hipEventDisableTiming) == hipSuccess;
        ok = ok && hipEventCreateWithFlags(&p->ev_join[0], hipEventDisableTiming) == hipSuccess;
        ok = ok && hipEventCreateWithFlags(&p->ev_join[1], hipEventDisableTiming) == hipSuccess;
        if (!ok) (void)hipGetLastError();
        p->side_ok = ok ? 1 : 0;
    }
}

extern "C" {

void hcspmm_default_options(hcspmm_options* opt)
{
    if (!opt) return;
    memset(opt, 0, sizeof *opt);
    opt->struct_size = (int32_t)sizeof *opt;
    opt->window_rows = kH;
    opt->route_mode = HCSPMM_ROUTE_HYBRID;
    opt->mfma_dtype = HCSPMM_F32;
    opt->d_hint = 0;
    opt->use_custom_selector = 0;
}

hcspmm_status hcspmm_default_selector(int32_t mfma_dtype, int32_t d_hint, int64_t nnz, int64_t* coef)
{
    if (!coef) { set_error("coef is NULL"); return HCSPMM_EINVAL; }
    if (nnz < 0) { set_error("nnz is negative"); return HCSPMM_EINVAL; }
    if (!lookup_selector(mfma_dtype, d_hint, nnz, coef)) { set_error("unknown mfma_dtype %d", mfma_dtype); return HCSPMM_EINVAL; }
    return HCSPMM_OK;
}

hcspmm_status hcspmm_prepare(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t* d_rowptr,
                             const int32_t* d_colind, const float* d_vals, const hcspmm_options* opt, void* stream,
                             hcspmm_plan** out_plan)
{
    if (!out_plan) { set_error("out_plan is NULL"); return HCSPMM_EINVAL; }
    *out_plan = nullptr;
    if (n_rows < 0 || n_cols < 1 || nnz < 0) { set_error("negative size or n_cols < 1"); return HCSPMM_EINVAL; }
    if (n_cols >= (1 << 27)) { set_error("n_cols must be below 2^27"); return HCSPMM_EUNSUPPORTED; }
    if (nnz >= ((int64_t)1 << 31)) { set_error("nnz must be below 2^31"); return HCSPMM_EUNSUPPORTED; }
    if (!d_rowptr || (nnz > 0 && (!d_colind || !d_vals))) { set_error("NULL CSR array"); return HCSPMM_EINVAL; }
    hcspmm_options o;
    hcspmm_default_options(&o);
    if (opt) {
        if (opt->struct_size != (int32_t)sizeof(hcspmm_options)) { set_error("options.struct_size mismatch"); return HCSPMM_EINVAL; }
        o = *opt;
    }
    if (o.window_rows != kH) { set_error("only window_rows = 16 is implemented"); return HCSPMM_EUNSUPPORTED; }
    if (o.route_mode < 0 || o.route_mode > 3) { set_error("bad route_mode"); return HCSPMM_EINVAL; }
    if (o.mfma_dtype < 0 || o.mfma_dtype > 2) { set_error("bad mfma_dtype"); return HCSPMM_EINVAL; }
    if (o.d_hint < 0) { set_error("bad d_hint"); return HCSPMM_EINVAL; }
    if (o.update_fusion < 0 || o.update_fusion > 2) { set_error("bad update_fusion"); return HCSPMM_EINVAL; }
    if (o.matrix_kernels < 0 || o.matrix_kernels > 2) { set_error("bad matrix_kernels"); return HCSPMM_EINVAL; }
    hcspmm_plan* p = new (std::nothrow) hcspmm_plan();
    if (!p) { set_error("host allocation failed"); return HCSPMM_EALLOC; }
    hcspmm_status st = init_plan_header(p, n_rows, n_cols, nnz, d_rowptr, d_colind, d_vals, o);
    if (st != HCSPMM_OK) { delete p; return st; }
    st = build_plan(p, static_cast<hipStream_t>(stream));
    if (st != HCSPMM_OK) { delete p; return st; }
    if ((st = reserve_row_sums(p, 0)) != HCSPMM_OK) { free_plan_arrays(p); delete p; return st; }
    setup_side_streams(p);
    *out_plan = p;
    return HCSPMM_OK;
}

hcspmm_status hcspmm_plan_update(hcspmm_plan* plan, int64_t nnz, const int32_t* d_rowptr, const int32_t* d_colind,
                                 const float* d_vals, const int32_t* h_changed_rows, int32_t n_changed, void* stream)
{
    if (!plan) { set_error("plan is NULL"); return HCSPMM_EINVAL; }
    if (nnz < 0 || n_changed < 0 || (n_changed > 0 && !h_changed_rows)) { set_error("negative size or NULL row list"); return HCSPMM_EINVAL; }
    if (nnz >= ((int64_t)1 << 31)) { set_error("nnz must be below 2^31"); return HCSPMM_EUNSUPPORTED; }
    if (!d_rowptr || (nnz > 0 && (!d_colind || !d_vals))) { set_error("NULL CSR array"); return HCSPMM_EINVAL; }
    hipStream_t s = static_cast<hipStream_t>(stream);
    // the windows that hold a changed row, ascending and distinct
    std::vector<int32_t> touched;
    {
        std::vector<uint8_t> mark((size_t)plan->W, 0);
        for (int32_t i = 0; i < n_changed; ++i) {
            const int32_t r = h_changed_rows[i];
            if (r < 0 || r >= plan->n_rows) { set_error("changed row %d is outside the matrix", r); return HCSPMM_EINVAL; }
            mark[(size_t)(r / kH)] = 1;
        }
        for (int32_t w = 0; w < plan->W; ++w)
            if (mark[(size_t)w]) touched.push_back(w);
    }
    hcspmm_plan fresh;
    hcspmm_status st = init_plan_header(&fresh, plan->n_rows, plan->n_cols, nnz, d_rowptr, d_colind, d_vals, plan->opt);
    if (st != HCSPMM_OK) return st;
    // a plan that is updated keeps the device blocks of its updates (see BlockCache)
    if (!plan->cache) plan->cache = new (std::nothrow) BlockCache;
    fresh.cache = plan->cache;
    PlanCarry carry{plan->ncols, touched.data(), (int32_t)touched.size()};
    // The counts of untouched windows are carried over whenever the old plan has them and fewer than an eighth of
    // the windows changed (beyond that the list-driven passes cost as much as the plain ones); otherwise this is a
    // preparation from scratch.
    const bool incremental = plan->features_complete && plan->nnz > 0 && !touched.empty() && 8 * (int64_t)touched.size() < plan->W &&
                             !(plan->opt.route_mode == HCSPMM_ROUTE_ALL_CSR);
    if (incremental) {
        // (a plan with an unsorted row somewhere does not say where: its structure is not carried)
        if (plan->n_mfma > 0 && plan->erc && plan->wcols && plan->rows_sorted && !plan->scalar_exec) {
            carry.old_route = plan->route; carry.old_wptr = plan->wptr; carry.old_nnzw = plan->nnzw;
            carry.old_wcols = plan->wcols; carry.old_erc = plan->erc;
        }
    }
    const bool nothing_changed = touched.empty() && nnz == plan->nnz && plan->features_complete;
    if (nothing_changed) {
        HC_HIP(hipStreamSynchronize(s));                         // calls that still use the old arrays are done
        // same structure: only the borrowed pointers move
        plan->rowptr = d_rowptr; plan->colind = d_colind; plan->vals = d_vals;
        return HCSPMM_OK;
    }
    // (build_plan waits for the stream before it returns a plan, so calls that use the old arrays are done by then.  Waiting for them here as
    // well left the GPU idle while this call allocates and launches: 1,000 rows of 169,343 changed behind a product, twice: 328 -> 297 us.)
    st = build_plan(&fresh, s, incremental ? &carry : nullptr);
    if (st != HCSPMM_OK) return st;                              // the old plan is untouched and still valid for the old arrays
    if ((st = reserve_row_sums(&fresh, plan->acc_rows_elems)) != HCSPMM_OK) { free_plan_arrays(&fresh); return st; }
    // the new tables replace the old ones; streams, events and the lazily sized scratch buffers stay
    fresh.partial = plan->partial; fresh.partial_elems = plan->partial_elems;
    fresh.tile_partial = plan->tile_partial; fresh.tile_partial_elems = plan->tile_partial_elems;
    if (!fresh.acc_rows) { fresh.acc_rows = plan->acc_rows; fresh.acc_rows_elems = plan->acc_rows_elems; plan->acc_rows = nullptr; }
    plan->partial = nullptr; plan->tile_partial = nullptr;
    free_plan_arrays(plan);
    fresh.side_ok = plan->side_ok;
    fresh.side[0] = plan->side[0]; fresh.side[1] = plan->side[1];
    fresh.ev_fork = plan->ev_fork; fresh.ev_join[0] = plan->ev_join[0]; fresh.ev_join[1] = plan->ev_join[1];
    *plan = fresh;
    setup_side_streams(plan);
    if (plan->cache) plan->cache->end_of_update();
    return HCSPMM_OK;
}

hcspmm_status hcspmm_plan_info(const hcspmm_plan* p, hcspmm_plan_info_t* info)
{
    if (!p || !info) { set_error("NULL argument"); return HCSPMM_EINVAL; }
    if (!p->features_complete) {
        const hcspmm_status st = complete_condensed(const_cast<hcspmm_plan*>(p), true);
        if (st != HCSPMM_OK) return st;
    }
    memset(info, 0, sizeof *info);
    info->window_rows = p->H; info->n_rows = p->n_rows; info->n_cols = p->n_cols; info->nnz = p->nnz;
    info->n_windows = p->W; info->total_ncols = p->total_ncols;
    info->n_mfma_windows = p->n_mfma; info->n_csr_windows = p->n_csr; info->nnz_mfma = p->nnz_mfma;
    info->route_mode = p->opt.route_mode; info->mfma_dtype = p->opt.mfma_dtype; info->d_hint = p->opt.d_hint;
    for (int i = 0; i < 3; ++i) info->sel_coef[i] = p->coef[i];
    info->device_bytes = p->device_bytes + (p->partial_elems + p->tile_partial_elems + p->acc_rows_elems) * (int64_t)sizeof(float);
    info->n_short_rows = p->n_short; info->n_long_rows = p->n_long_rows; info->n_segments = p->n_segs;
    info->n_mid_rows = p->n_mid;
    info->nnz_long = p->nnz_long;
    // (launch tables: none of the matrix path's kernels runs where the scalar path has taken its windows over)
    info->n_mfma_small = p->scalar_exec ? 0 : p->n_mfma_small;
    info->n_mfma_big = p->scalar_exec ? 0 : p->n_mfma_mid + p->n_mfma_big;
    info->n_runs = p->runs_ok ? p->n_runs : 0;
    info->n_run_slices = p->runs_ok ? p->n_run_slices : 0;
    info->run_union_cols = p->runs_ok ? p->run_union_cols : 0;
    return HCSPMM_OK;
}

hcspmm_status hcspmm_plan_export(const hcspmm_plan* p, int32_t* ncols, int32_t* nnzw, uint8_t* route, int64_t* wptr,
                                 int32_t* wcols, int32_t* ecol, int32_t* mfma_windows, int32_t* csr_windows)
{
    if (!p) { set_error("plan is NULL"); return HCSPMM_EINVAL; }
    HC_HIP(hipDeviceSynchronize());
    if (!p->features_complete || ((wcols || ecol) && !p->condensed_complete)) {
        const hcspmm_status st = complete_condensed(const_cast<hcspmm_plan*>(p), !(wcols || ecol));
        if (st != HCSPMM_OK) return st;
    }
    const size_t W = (size_t)p->W;
    if (ncols && W) HC_HIP(hipMemcpy(ncols, p->ncols, W * 4, hipMemcpyDeviceToHost));
    if (nnzw && W) HC_HIP(hipMemcpy(nnzw, p->nnzw, W * 4, hipMemcpyDeviceToHost));
    if (route && W) HC_HIP(hipMemcpy(route, p->route, W, hipMemcpyDeviceToHost));
    if (wptr) HC_HIP(hipMemcpy(wptr, p->wptr, (W + 1) * 8, hipMemcpyDeviceToHost));
    if (wcols && p->total_ncols) HC_HIP(hipMemcpy(wcols, p->wcols, (size_t)p->total_ncols * 4, hipMemcpyDeviceToHost));
    if (ecol && p->nnz) {
        HC_HIP(hipMemcpy(ecol, p->erc, (size_t)p->nnz * 4, hipMemcpyDeviceToHost));
        for (int64_t k = 0; k < p->nnz; ++k) ecol[k] >>= 4;    // drop the packed row-in-window
    }
    if ((mfma_windows || csr_windows) && W) {
        std::vector<uint8_t> h_route(W);
        HC_HIP(hipMemcpy(h_route.data(), p->route, W, hipMemcpyDeviceToHost));
        for (int32_t w = 0; w < p->W; ++w) {
            int32_t*& list = h_route[(size_t)w] ? mfma_windows : csr_windows;
            if (list) *list++ = w;
        }
    }
    return HCSPMM_OK;
}

hcspmm_status hcspmm_plan_export_runs(const hcspmm_plan* p, int32_t* run_nu, int32_t* ucols, int32_t* wslot)
{
    if (!p) { set_error("plan is NULL"); return HCSPMM_EINVAL; }
    if (!p->runs_ok) { set_error("the plan has no run table (prepare with matrix_kernels = HCSPMM_MATRIX_RUNS)"); return HCSPMM_EINVAL; }
    HC_HIP(hipDeviceSynchronize());
    std::vector<RunDesc> h_runs((size_t)p->n_runs);
    HC_HIP(hipMemcpy(h_runs.data(), p->runs, h_runs.size() * sizeof(RunDesc), hipMemcpyDeviceToHost));
    int64_t at = 0;
    for (const RunDesc& r : h_runs) {
        if (run_nu) run_nu[&r - h_runs.data()] = r.nu;
        if (ucols && r.nu > 0) HC_HIP(hipMemcpy(ucols + at, p->ucols + r.up, (size_t)r.nu * sizeof(int32_t), hipMemcpyDeviceToHost));
        at += r.nu;
    }
    if (wslot && p->total_ncols > 0) HC_HIP(hipMemcpy(wslot, p->wslot, (size_t)p->total_ncols * sizeof(int32_t), hipMemcpyDeviceToHost));
    return HCSPMM_OK;
}

static hcspmm_status check_dense(const char* name, const void* ptr, int64_t ld, int32_t width)
{
    if (!ptr) { set_error("%s is NULL", name); return HCSPMM_EINVAL; }
    if (ld < width) { set_error("leading dimension of %s (%lld) is smaller than its width (%d)", name, (long long)ld, width); return HCSPMM_EINVAL; }
    return HCSPMM_OK;
}

static hcspmm_status spmm_impl(const hcspmm_plan* plan, const void* d_X, int64_t ldx, int32_t d, int32_t x_dtype,
                               void* d_Y, int64_t ldy, int32_t y_dtype, void* stream, hipEvent_t* ev,
                               bool static_scratch = false);

hcspmm_status hcspmm_spmm(const hcspmm_plan* plan, const void* d_X, int64_t ldx, int32_t d, int32_t x_dtype, void* d_Y,
                          int64_t ldy, int32_t y_dtype, void* stream)
{
    return spmm_impl(plan, d_X, ldx, d, x_dtype, d_Y, ldy, y_dtype, stream, nullptr);
}

hcspmm_status hcspmm_spmm_timed(const hcspmm_plan* plan, const void* d_X, int64_t ldx, int32_t d, int32_t x_dtype,
                                void* d_Y, int64_t ldy, int32_t y_dtype, void* stream, hcspmm_stage_times* times)
{
    if (!times) { set_error("times is NULL"); return HCSPMM_EINVAL; }
    memset(times, 0, sizeof *times);
    hipEvent_t ev[5];
    int made = 0;
    hcspmm_status st = HCSPMM_OK;
    for (; made < 5; ++made)
        if (hipEventCreate(&ev[made]) != hipSuccess) { (void)hipGetLastError(); set_error("hipEventCreate failed"); st = HCSPMM_EHIP; break; }
    if (st == HCSPMM_OK) st = spmm_impl(plan, d_X, ldx, d, x_dtype, d_Y, ldy, y_dtype, stream, ev);
    if (st == HCSPMM_OK && plan->n_rows > 0) {
        if (hipEventSynchronize(ev[4]) != hipSuccess) { (void)hipGetLastError(); set_error("hipEventSynchronize failed"); st = HCSPMM_EHIP; }
        else {
            float* out[4] = {&times->ms_mfma_big, &times->ms_mfma_small, &times->ms_csr, &times->ms_csr_reduce};
            for (int i = 0; i < 4; ++i) (void)hipEventElapsedTime(out[i], ev[i], ev[i + 1]);
            (void)hipEventElapsedTime(&times->ms_total, ev[0], ev[4]);
        }
    }
    for (int i = 0; i < made; ++i) (void)hipEventDestroy(ev[i]);
    return st;
}

static hcspmm_status spmm_impl(const hcspmm_plan* plan, const void* d_X, int64_t ldx, int32_t d, int32_t x_dtype,
                               void* d_Y, int64_t ldy, int32_t y_dtype, void* stream, hipEvent_t* ev, bool static_scratch)
{
    if (!plan) { set_error("plan is NULL"); return HCSPMM_EINVAL; }
    if (d < 1 || d > (1 << 20)) { set_error("d must be in [1, 2^20]"); return HCSPMM_EINVAL; }
    if (x_dtype < 0 || x_dtype > 2 || y_dtype < 0 || y_dtype > 2) { set_error("bad dtype"); return HCSPMM_EINVAL; }
    if (plan->n_rows == 0) return HCSPMM_OK;
    hcspmm_status st;
    if ((st = check_dense("X", d_X, ldx, d)) != HCSPMM_OK) return st;
    if ((st = check_dense("Y", d_Y, ldy, d)) != HCSPMM_OK) return st;
    SpmmArgs a{};
    a.n_rows = plan->n_rows; a.n_cols = plan->n_cols; a.rowptr = plan->rowptr; a.colind = plan->colind; a.vals = plan->vals;
    a.X = d_X; a.ldx = ldx; a.d = d; a.x_dtype = x_dtype; a.Y = static_cast<float*>(d_Y); a.ldy = ldy; a.relu = 0;
    a.y_dtype = y_dtype;
    if (plan->n_mfma > 0 && !plan->scalar_exec && !mfma_shape_supported(a)) {
        set_error("16-bit X on the matrix path needs d, ldx and ldy to be multiples of 4 and 8-byte aligned X, 16-byte aligned Y");
        return HCSPMM_EUNSUPPORTED;
    }
    char* scratch_mem = nullptr;
    if (static_scratch) {
        const size_t need = spmm_scratch_bytes(plan, d, nullptr);
        if (need > kStaticScratchBytes) {
            set_error("this plan needs %zu bytes of scratch at d = %d, the static scratch array holds %zu; use hcspmm_spmm",
                      need, d, kStaticScratchBytes);
            return HCSPMM_EUNSUPPORTED;
        }
        if ((st = static_scratch_ptr(plan, &scratch_mem)) != HCSPMM_OK) return st;
    }
    return run_spmm(plan, a, static_cast<hipStream_t>(stream), ev, nullptr, false, scratch_mem, d <= plan->acc_width);
}

hcspmm_status hcspmm_spmm_noalloc(const hcspmm_plan* plan, const void* d_X, int64_t ldx, int32_t d, int32_t x_dtype,
                                  void* d_Y, int64_t ldy, int32_t y_dtype, void* stream)
{
    return spmm_impl(plan, d_X, ldx, d, x_dtype, d_Y, ldy, y_dtype, stream, nullptr, true);
}

size_t hcspmm_spmm_noalloc_scratch_limit(void) { return kStaticScratchBytes; }

size_t hcspmm_gcn_workspace_bytes(const hcspmm_plan* plan, int32_t d_in, int32_t d_out)
{
    (void)d_in;
    if (!plan || d_out < 1) return 0;
    size_t b = (size_t)plan->n_cols * (size_t)d_out * sizeof(float);
    return (b + 255) & ~(size_t)255;
}

hcspmm_status hcspmm_gemm_f32(int64_t m, int32_t k, int32_t n, const float* d_X, int64_t ldx, const float* d_W,
                              int64_t ldw, float* d_T, int64_t ldt, void* stream)
{
    if (m < 0 || k < 0 || n < 0) { set_error("negative size"); return HCSPMM_EINVAL; }
    if (m == 0 || n == 0) return HCSPMM_OK;
    hcspmm_status st;
    if (k > 0 && (st = check_dense("X", d_X, ldx, k)) != HCSPMM_OK) return st;
    if (k > 0 && (st = check_dense("W", d_W, ldw, n)) != HCSPMM_OK) return st;
    if ((st = check_dense("T", d_T, ldt, n)) != HCSPMM_OK) return st;
    HC_HIP(launch_gemm_f32(m, k, n, d_X, ldx, d_W, ldw, d_T, ldt, nullptr, 0, static_cast<hipStream_t>(stream)));
    return HCSPMM_OK;
}

// bytes from the first to the last element of a matrix with rows of w elements
static size_t extent_bytes(int64_t rows, int64_t ld, int64_t w, size_t element) { return rows > 0 ? (size_t)((rows - 1) * ld + w) * element : 0; }
static bool overlap(const void* a, size_t na, const void* b, size_t nb)
{
    return (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

static bool aggregate_first(const hcspmm_plan* plan, const SpmmArgs& a, int32_t d_out, size_t workspace);
static hcspmm_status aggregate_then_update(const hcspmm_plan* plan, const SpmmArgs& a, const float* W, int64_t ldw, int32_t d_out, void* Y,
                                           int64_t ldy, int32_t y_dtype, int32_t apply_relu, hipStream_t s);

hcspmm_status hcspmm_gcn_layer(const hcspmm_plan* plan, const void* d_X, int64_t ldx, int32_t d_in, const void* d_W,
                               int64_t ldw, int32_t d_out, void* d_Y, int64_t ldy, int32_t apply_relu,
                               void* d_workspace, size_t workspace_bytes, void* stream)
{
    return hcspmm_gcn_layer_ex(plan, d_X, ldx, d_in, d_W, ldw, d_out, d_Y, ldy, HCSPMM_F32, apply_relu, HCSPMM_F32, d_workspace,
                               workspace_bytes, stream);
}

hcspmm_status hcspmm_gcn_layer_ex(const hcspmm_plan* plan, const void* d_X, int64_t ldx, int32_t d_in, const void* d_W,
                                  int64_t ldw, int32_t d_out, void* d_Y, int64_t ldy, int32_t y_dtype, int32_t apply_relu,
                                  int32_t t_dtype, void* d_workspace, size_t workspace_bytes, void* stream)
{
    if (!plan) { set_error("plan is NULL"); return HCSPMM_EINVAL; }
    if (y_dtype != HCSPMM_F32 && y_dtype != HCSPMM_BF16 && y_dtype != HCSPMM_F16) { set_error("y_dtype %d is not a dtype code", y_dtype); return HCSPMM_EINVAL; }
    if (d_in < 1 || d_out < 1 || d_in > (1 << 20) || d_out > (1 << 20)) { set_error("d_in, d_out must be in [1, 2^20]"); return HCSPMM_EINVAL; }
    if (t_dtype != HCSPMM_F32 && t_dtype != HCSPMM_BF16 && t_dtype != HCSPMM_F16) { set_error("t_dtype %d is not a dtype code", t_dtype); return HCSPMM_EINVAL; }
    hcspmm_status st;
    if ((st = check_dense("X", d_X, ldx, d_in)) != HCSPMM_OK) return st;
    if ((st = check_dense("W", d_W, ldw, d_out)) != HCSPMM_OK) return st;
    if ((st = check_dense("Y", d_Y, ldy, d_out)) != HCSPMM_OK) return st;
    const size_t need = hcspmm_gcn_workspace_bytes(plan, d_in, d_out);      // sized for fp32 T; 16-bit T uses half of it
    if (!d_workspace || workspace_bytes < need) { set_error("workspace too small: need %zu bytes", need); return HCSPMM_EINVAL; }
    if (((uintptr_t)d_workspace & 255) != 0) { set_error("workspace must be 256-byte aligned"); return HCSPMM_EINVAL; }
    hipStream_t s = static_cast<hipStream_t>(stream);
    SpmmArgs a{};
    a.n_rows = plan->n_rows; a.n_cols = plan->n_cols; a.rowptr = plan->rowptr; a.colind = plan->colind; a.vals = plan->vals;
    a.X = d_workspace; a.ldx = d_out; a.d = d_out; a.x_dtype = t_dtype; a.Y = static_cast<float*>(d_Y); a.ldy = ldy;
    a.relu = apply_relu ? 1 : 0;
    a.y_dtype = y_dtype;
    if (t_dtype != HCSPMM_F32 && plan->n_mfma > 0 && !plan->scalar_exec && !mfma_shape_supported(a)) {
        set_error("the matrix path with 16-bit T needs d_out a multiple of 4 and 16-byte aligned Y rows");
        return HCSPMM_EUNSUPPORTED;
    }
    // The order of the two products depends on X's base and pitch; scratch follows from the shapes alone and serves both orders
    // (the other order's rows are no wider), so that after one call any call of the same shapes allocates nothing.
    hcspmm_plan* p = const_cast<hcspmm_plan*>(plan);
    if (plan->n_rows > 0 && (st = reserve_scratch(p, d_out, s)) != HCSPMM_OK) return st;
    if (plan->n_rows > 0 && panel_sums_needed(plan, a) && (st = reserve_panel_sums(p, d_out, s)) != HCSPMM_OK) return st;
    // (X W in the workspace is complete before anything is stored to Y, so that Y may lie over X or W; the other order reads both
    // while it stores)
    const size_t y_size = extent_bytes(plan->n_rows, ldy, d_out, y_dtype == HCSPMM_F32 ? 4 : 2);
    const bool apart = !overlap(d_Y, y_size, d_X, extent_bytes(plan->n_cols, ldx, d_in, 4)) && !overlap(d_Y, y_size, d_W, extent_bytes(d_in, ldw, d_out, 4));
    if (t_dtype == HCSPMM_F32 && apart) {
        SpmmArgs z = a;
        z.X = d_X; z.ldx = ldx; z.d = d_in; z.Y = static_cast<float*>(d_workspace); z.ldy = d_in; z.relu = 0; z.y_dtype = HCSPMM_F32;
        if (aggregate_first(plan, z, d_out, need))
            return aggregate_then_update(plan, z, static_cast<const float*>(d_W), ldw, d_out, d_Y, ldy, y_dtype, apply_relu, s);
    }
    HC_HIP(launch_gemm_f32_out(plan->n_cols, d_in, d_out, static_cast<const float*>(d_X), ldx,
                               static_cast<const float*>(d_W), ldw, d_workspace, d_out, t_dtype, 0, s));
    if (plan->n_rows == 0) return HCSPMM_OK;
    return run_spmm(plan, a, s, nullptr, nullptr, false, nullptr, true);
}

// Which windows keep their aggregated rows on chip for the update, when the caller leaves the choice to the library.
//  * A graph so small that launches dominate: all of them, in one pass (2,708 rows: 64 -> 128 columns 8.2 us against 9.9 us
//    with the product apart; at 16,934 rows it is 28.6 us against 19.7 us, and the line moves with the width).
//  * A large aggregation is bound by what it fetches from behind L2 and hides the product, and the round trip of the
//    aggregated rows is what is left to save (apart / in one pass, us): 1 M rows of 60, 32 -> 32: 910 / 883, 64 -> 64: 1946 /
//    1892, 128 -> 128: 4221 / 3908; 2.4 M of 51: 2236 / 2165, 4652 / 4415, 9374 / 8658; but 2.4 M of 20: 972 / 1027, 1911 /
//    2209.  A product of 128 x 128 or more is large enough to be hidden earlier: 500,000 of 60: 1926 / 1814, 2.4 M of 20: 4245 /
//    4081, 300,000 of 60: 1040 / 1027; f16 470,000 of 57: 896 / 859.  When the pass has to store the aggregated rows all the same (the weight gradient reads
//    them) it takes 40 non-zeros per row: 1 M of 40, 128 -> 128: 3268 / 3083, 2.4 M of 20: 4879 / 4945.
//  * Otherwise the scalar path's rows go through the workspace: its own kernel with column slices and a whole product
//    are ahead of tiles of 16 rows that wait for their longest row (169,343 rows, 32 -> 32: 73 us against 47 us, 128 -> 128:
//    195 us against 175 us).
//  * The wave-per-window matrix kernel multiplies its tile while other waves gather, unless the multiplication outweighs the
//    gather it hides behind (apart / in the windows; communities of degree 51, 131,072 rows: 64 -> 256: 124 / 108 us, 128 ->
//    128: 153 / 153 us, 128 -> 160: 170 / 181 us, 256 -> 80: 308 / 349 us; of degree 20: 128 -> 64 74 / 68 us, 192 -> 128 133 /
//    153 us); few windows do not hide it (16,384 rows, 96 -> 256: 32 / 40 us).  W of an odd width is read value by value there and
//    hides behind no gather of rows of 96 columns and more (bf16, 299,968 of 37: 144 -> 97 278 / 498 us, 96 -> 33 130 / 154; 70,016
//    of 42: 128 -> 47 50 / 52; fp32, 131,072 of 17: 96 -> 67 85 / 115).
enum UpdatePlace { kUpdateApart, kUpdateInWindows, kUpdateEverywhere };
static UpdatePlace update_place(const hcspmm_plan* plan, int32_t agg_width, int32_t out_width, int32_t x_dtype, bool keep_z)
{
    const int64_t product = (int64_t)agg_width * out_width;
    const bool windows = !plan->scalar_exec && 2 * plan->n_mfma_small >= plan->W;
    if (plan->n_panels < 2 && 4 * (int64_t)plan->n_rest < plan->n_rows) {
        const double degree = plan->n_rows > 0 ? (double)plan->nnz / plan->n_rows : 0.0;
        if ((int64_t)plan->n_rows * agg_width <= 200000 && plan->n_rows <= 8192) return kUpdateEverywhere;
        // (the pass reads a row with all lanes of its form at once; 16-bit rows that leave some of them idle are better cut
        // into column slices: 2.4 M of 51, f16, 208 -> 183: 10.7 ms apart, 12.3 ms in one pass)
        const bool f32 = x_dtype == HCSPMM_F32, full = (agg_width & (agg_width - 1)) == 0;
        if (!windows && (f32 || full)) {
            if (plan->n_rows >= 1000000 && degree >= 50.0) return kUpdateEverywhere;
            if (product >= 16384 && plan->n_rows >= 300000 && plan->nnz >= 16000000 && (full || agg_width <= 128) &&
                degree >= (!f32 ? 50.0 : keep_z ? 40.0 : 0.0))
                return kUpdateEverywhere;
        }
    }
    if (agg_width >= 96 && out_width % 2 != 0) return kUpdateApart;
    return windows && product <= (plan->n_mfma_small >= 4096 ? 16384 : 12288) ? kUpdateInWindows : kUpdateApart;
}

// 128-byte lines that a row of w elements of es bytes touches on average, by what its base and pitch are multiples of
static double row_lines(const void* base, int64_t ld, int32_t w, int es)
{
    const uint64_t all = (uint64_t)(uintptr_t)base | (uint64_t)ld * (uint64_t)es | 128u;
    const double unit = (double)(all & (~all + 1));             // the largest power of two that divides both, 128 at most
    const double bytes = (double)w * es;
    return std::ceil(bytes / unit) * unit / 128.0 + (128.0 - unit) / 128.0;
}

// The form that a lane group reads a row of so many bytes in: up to 128, 256, 512 bytes, or more of them.
static int row_form(int64_t bytes) { return bytes <= 128 ? 0 : bytes <= 256 ? 1 : bytes <= 512 ? 2 : 3; }
// Values per load, by what rows and base are multiples of.
static int row_vector(const void* base, int64_t ld, int32_t w)
{
    const uint64_t all = (uint64_t)(uintptr_t)base / 4 | (uint64_t)ld | (uint64_t)w;
    return all % 4 == 0 ? 4 : all % 2 == 0 ? 2 : 1;
}

// Whether Y = act((A X) W) is computed as act(A (X W)): the same sums in fp32, associated the other way.  Where W makes rows
// shorter the gather, which is most of the call, then reads rows of d_out instead of d_in columns, and one trip of the rows
// through memory (X in, X W out) takes the place of the aggregated rows' (out and in again).  In this order / X W first, us:
// 169,343 rows of 14, fp32: 64 -> 32 columns 85 / 51, 128 -> 64 144 / 93, 256 -> 128 380 / 232; 400,000 of 40, 128 -> 64: 975 /
// 498; 1 M of 60 (in one pass with the product): 3825 / 2274; 131,072 in communities, 128 -> 64: 96 / 64.
//
// What counts is the share of the lines that a gathered row still touches, and where X stays in the L2s also whether the row takes
// fewer loads of a lane group (row_form).  Power laws, fp32: 24,000 rows of 15, 160 -> 128 (.80, fewer loads) 39 / 35, 144 -> 115
// (.91, fewer) 47 / 45, but 128 -> 96 (.75, as many) 27 / 31, 192 -> 160 (.83, as many) 47 / 48; 41,000 of 15: 176 -> 140 (.88, as
// many) 79 / 83; 60,000 of 15: 192 -> 160 108 / 99.  So: up to .6 always, up to .92 with fewer loads or from 24 MB of X on (57,140 of
// 74, 118 -> 96, .65: 222 / 126; 48 MB where X W is off the 16-byte pieces and X on them), up to .7 where there is much to gather
// (34,396 of 85, 18 -> 16: 30.7 / 25.2); and with some work to save (16,934 of 6, 224 -> 80: 26.6 / 27.4; 3,780 of 32, bf16, 224 ->
// 80: 18 / 20).
// On the matrix path the walks over the windows count as well, each of which takes up to four groups of 16 loads, of one, two or
// four values by what rows are multiples of (mfma_walks).  More walks than for X and half of the lines are too many (in communities:
// 11,008, 80 -> 33, .67: 25 / 32, 14,336, 80 -> 43, .77: 26 / 33); fewer walks, or as many with fewer loads, are ahead whatever the
// lines (671,825 of 18, 160 -> 93, .78: 835 / 685; 134,400 of 53, 74 -> 55, .83: 174 / 108), and so are larger pieces (76,352 of 57,
// 117 -> 112, .86: 135 / 96); as many walks and loads up to .8 where most windows are there (level to 1.2 times as fast).
//
// X W is held in fp32, so that 16-bit rows have to become half as long for the same bytes: 169,343 of 14, bf16, 128 -> 64: 98 / 80,
// 128 -> 48: 95 / 75 (but 128 -> 72: 104 / 119); 400,000 of 40, f16, 256 -> 96: 974 / 693.  Up to .83 of the lines, and as many
// lines for rows of a line and more that come from behind L2 and go through the workspace (bf16: 169,343 of 14, 128 -> 64 above,
// 156,832 of 32, 64 -> 32: 53 / 49; but 46,367 of 7, 64 -> 32: 15.9 / 17.8, 102,206 of 16, 48 -> 13 (.92): 33 / 34, 81,692 of 35, 52
// -> 11, off the 16-byte pieces: 36 / 41), if no window runs on the matrix path or the loads are fewer (1 M of 60, bf16, 128 -> 64,
// 3,145 windows there: 1885 / 2075; 2 M of 20, 160 -> 57: 2712 / 2201).  Matrix-path windows fetch a 16-bit row once per window and multiply on chip: 67,520 in communities, bf16, 80 -> 32:
// 41 / 52, 32,128, f16, 128 -> 32: 25 / 29; rows of more than 256 bytes still gain where they are many (88,576, f16, 232 -> 14: 70 /
// 47; but 11,008, 176 -> 32: 17.6 / 18.3), and so do windows of few non-zeros with 48 MB of X (299,968 rows of 21, bf16, 112 -> 16:
// 109 / 96, but of 37, 68 -> 16: 106 / 115).
// What the other order refuses stays refused, and nothing is allocated that it would not have allocated.
static bool update_before(const hcspmm_plan* plan, const SpmmArgs& a, int32_t d_out, int32_t y_dtype, size_t workspace)
{
    if (plan->opt.update_fusion != HCSPMM_UPDATE_AUTO) return false;
    if (d_out > a.d) return false;      // (a row off the lines may touch more of them and be narrower: partial sums grow with the width)
    if (plan->n_cols > plan->n_rows || (size_t)plan->n_cols * d_out * sizeof(float) > workspace) return false;
    const bool f32 = a.x_dtype == HCSPMM_F32;
    if (!f32 && !gemm_x16_usable(a.X, a.ldx)) return false;
    const bool matrix = plan->n_mfma > 0 && !plan->scalar_exec, windows = matrix && 2 * plan->n_mfma_small >= plan->W;
    if (matrix && !mfma_shape_supported(a)) return false;
    // (sums between panels that the plan was made with, not what an earlier call may have left: the order must not depend on that)
    if (plan->n_panels > 1 && y_dtype != HCSPMM_F32 && d_out > plan->acc_width) return false;
    const int es = f32 ? 4 : 2;
    const double share = row_lines(nullptr, d_out, d_out, 4) / row_lines(a.X, a.ldx, a.d, es);
    const double x_mb = (double)plan->n_cols * a.d * es / (1 << 20);
    const bool apart = update_place(plan, a.d, d_out, a.x_dtype, false) == kUpdateApart, many = plan->n_rows >= 40000;
    if ((!many && plan->nnz < (share <= 0.5 ? 100000 : 150000)) || (plan->n_rows <= 8192 && !apart)) return false;
    if (f32) {
        const bool fewer = row_form(4 * (int64_t)d_out) < row_form(4 * (int64_t)a.d);
        const int before = row_vector(a.X, a.ldx, a.d), after = row_vector(nullptr, d_out, d_out);
        if (matrix) {
            const int walks = mfma_walks(nullptr, d_out, d_out) - mfma_walks(a.X, a.ldx, a.d);
            if (walks > 0 && share > 0.5) return false;
            if (share <= (walks < 0 || fewer ? 1.0 : after > before ? 0.92 : windows ? 0.8 : 0.0)) return true;
        }
        if (share <= 0.6) return d_out < a.d || plan->nnz >= 40 * (int64_t)plan->n_rows;    // (seldom for a better place of rows alone)
        if (share > 0.92) return false;
        if (!matrix && (fewer || (share <= 0.7 && after >= before && plan->nnz >= 80 * (int64_t)plan->n_rows))) return true;
        return plan->n_panels < 2 && x_mb >= (matrix || after < before ? 48.0 : 24.0);
    }
    if (matrix && (windows || !many)) {
        if (windows && x_mb >= 48.0 && plan->nnz < 24 * (int64_t)plan->n_rows) return share <= 0.6;
        return 2 * a.d > 256 && share <= 0.5 && (many || !windows);
    }
    const bool fewer = row_form(4 * (int64_t)d_out) < row_form(2 * (int64_t)a.d), pieces = d_out % 4 == 0 || fewer;
    return share <= (pieces ? 0.83 : 0.6) || (share <= 1.0 && pieces && (!matrix || fewer) && 2 * a.d >= 128 && x_mb >= 16.0 && plan->n_panels < 2 && apart);
}

// Y = act((A X) W) in that order, A X (a.Y, where it reaches memory) in the caller's workspace.
static hcspmm_status aggregate_then_update(const hcspmm_plan* plan, const SpmmArgs& a, const float* W, int64_t ldw, int32_t d_out, void* Y,
                                           int64_t ldy, int32_t y_dtype, int32_t apply_relu, hipStream_t s)
{
    const UpdatePlace place = plan->opt.update_fusion == HCSPMM_UPDATE_FUSED   ? kUpdateEverywhere
                              : plan->opt.update_fusion == HCSPMM_UPDATE_SPLIT ? kUpdateApart
                                                                               : update_place(plan, a.d, d_out, a.x_dtype, false);
    if (place != kUpdateApart && update_fusable(a)) {
        const UpdateArgs u{W, ldw, d_out, static_cast<float*>(Y), ldy, apply_relu ? 1 : 0, 0, nullptr, 0, y_dtype};
        return run_spmm(plan, a, s, nullptr, &u, place == kUpdateInWindows);
    }
    const hcspmm_status st = run_spmm(plan, a, s);
    if (st != HCSPMM_OK) return st;
    HC_HIP(launch_gemm_f32_out(plan->n_rows, a.d, d_out, a.Y, a.ldy, W, ldw, Y, ldy, y_dtype, apply_relu ? 1 : 0, s));
    return HCSPMM_OK;
}

// Whether the layer Y = act(A (X W)) is computed as act((A X) W), T = X W being asked for in fp32: the same trade as in
// update_before the other way.  Where W makes rows longer, rows of X are what a gather should read, and the aggregated rows' trip
// through memory is shorter than that of X W (or stays on chip, see update_place).  X W first / this order, fp32, us: power laws
// of 615,315 rows of 97, 32 -> 144 columns: 5923 / 1510; 66,756 of 161, 40 -> 188: 863 / 172; 58,920 of 40, 105 -> 176: 202 / 142;
// 371,268 of 6, 56 -> 112: 227 / 163; communities, 114,816 of 58, 112 -> 160: 223 / 140.
//
// The lines of a gathered row and its loads decide, as there: up to .7 of the lines (.6 where rows of X are off the 16-byte pieces
// and take as many loads: 72,512 in communities, 9 -> 27, .69: 34 / 37); up to .92 with fewer loads of a lane group, for rows of X W
// of more than a line that are read in no larger pieces or have up to 128 columns (133,729 of 56, 33 -> 50, .80: 218 / 163; 112,597
// of 359, 80 -> 112, .75: 1643 / 1097; 12,942 of 23, 160 -> 224, .71: 41 / 36; but 58,368 in communities, 14 -> 24, .92: 28 / 35;
// 30,214 of 36, 143 -> 176, .91: 87 / 94; 20,680 of 137, 191 -> 240, .87: 202 / 218), or from 48 MB of X W on, where no slices of a
// line stand against rows off the lines (56,233 of 79, 156 -> 224, .82: 347 / 403); as many lines where one holds the row of either and it is clearly shorter and read in whole
// vectors (142,285 of 16, 8 -> 16: 35.0 / 27.0; but 85,184 of 39, 40 -> 64, two lines: 50 / 52; 75,504 of 63, 48 -> 64: 96 / 98).
// Rows of X that are read in larger pieces than those of X W are ahead up to .92 (150,939 of 133, 24 -> 30, .91: 386 / 290).
// On the matrix path the walks over the windows decide as there (299,968 in communities, 160 -> 223, .63: 876 / 676; 16,192, 51 -> 69,
// .82: 36.5 / 21.2; 1.7 M of 14, few windows, 63 -> 170: 3880 / 2111; but more walks: 3,008 in communities, 37 -> 128, .53: 21 / 26,
// 70,144, 41 -> 80, .75: 80 / 108).  As many walks and loads pay up to .8, where most windows are there up to .6, .67 with the product
// in them (larger pieces up to .92: 11,264, 160 -> 218, .65: 58 / 50; 54,400, 144 -> 256, .62: 135 / 140; 174,848, in the windows, 96 -> 112, .75: 169 / 178, 121,344, 64 -> 80, .67: 111 / 92).
// The one pass over a few thousand rows walks a hub's non-zeros in one lane group: where more than one row in 48 is no short one it
// takes 128 MB less to gather to be ahead (2,170 rows of 60, 32 -> 96: 12.2 / 19.9, 3,376 of 80, 32 -> 96: 15.7 / 20.0, 3,862 of
// 163, 48 -> 96: 23.9 / 29.1; 6,850 of 58, 16 -> 113: 24.8 / 18.6).
static bool aggregate_first(const hcspmm_plan* plan, const SpmmArgs& a, int32_t d_out, size_t workspace)
{
    if (plan->opt.update_fusion != HCSPMM_UPDATE_AUTO || plan->n_rows == 0 || a.d > d_out) return false;
    if ((size_t)plan->n_rows * a.d * sizeof(float) > workspace) return false;
    const bool matrix = plan->n_mfma > 0 && !plan->scalar_exec, windows = matrix && 2 * plan->n_mfma_small >= plan->W;
    if (matrix && !mfma_shape_supported(a)) return false;
    const UpdatePlace place = update_fusable(a) ? update_place(plan, a.d, d_out, HCSPMM_F32, false) : kUpdateApart;
    const double share = row_lines(a.X, a.ldx, a.d, 4) / row_lines(nullptr, d_out, d_out, 4);
    const bool hubs = 48 * ((int64_t)plan->n_mid + plan->n_segs) > plan->n_rows;
    if (place == kUpdateEverywhere && plan->n_rows <= 8192 && hubs && plan->nnz * (d_out - a.d) * 4 < ((int64_t)128 << 20)) return false;
    const bool fewer = row_form(4 * (int64_t)a.d) < row_form(4 * (int64_t)d_out), on_lines = a.ldx % 32 == 0 && (uintptr_t)a.X % 128 == 0;
    const bool sliced = a.d > 128 && !on_lines && d_out % 32 == 0 && plan->nnz >= 40 * (int64_t)plan->n_rows;
    const int before = row_vector(nullptr, d_out, d_out), after = row_vector(a.X, a.ldx, a.d);
    const bool pieces = after == 4, long_rows = plan->n_rows > 8192 && 4 * (int64_t)d_out > 128;
    if (matrix) {
        const int walks = mfma_walks(a.X, a.ldx, a.d) - mfma_walks(nullptr, d_out, d_out);
        if (share <= (walks < 0 || (walks == 0 && fewer) ? 1.0 : 0.4)) return true;
        if (walks > 0) return false;
        if (share <= 0.92 && after > before) return true;
        if (windows) return share <= (place == kUpdateInWindows ? 0.67 : 0.6);
        if (share <= 0.8) return true;
    } else if (share <= 0.92 && (after > before || (long_rows && !sliced && (after == before || d_out <= 128)))) return true;
    if (share <= (fewer || pieces ? 0.7 : 0.6)) return true;
    if (share <= 0.92) {
        if (fewer) return true;
        return !sliced && plan->n_panels < 2 && (double)plan->n_cols * d_out * 4 >= 48.0 * (1 << 20);
    }
    return share <= 1.0 && pieces && 3 * (int64_t)a.d <= 2 * (int64_t)d_out && 4 * (int64_t)d_out <= 128;
}

size_t hcspmm_aggregate_update_workspace_bytes(const hcspmm_plan* plan, int32_t d_in, int32_t d_out)
{
    (void)d_out;
    if (!plan || d_in < 1) return 0;
    size_t b = (size_t)plan->n_rows * (size_t)d_in * sizeof(float);
    return (b + 255) & ~(size_t)255;
}

hcspmm_status hcspmm_aggregate_update(const hcspmm_plan* plan, const void* d_X, int64_t ldx, int32_t d_in,
                                      int32_t x_dtype, const void* d_W, int64_t ldw, int32_t d_out, void* d_Y,
                                      int64_t ldy, int32_t y_dtype, int32_t apply_relu, void* d_workspace,
                                      size_t workspace_bytes, void* stream)
{
    if (!plan) { set_error("plan is NULL"); return HCSPMM_EINVAL; }
    if (y_dtype != HCSPMM_F32 && y_dtype != HCSPMM_BF16 && y_dtype != HCSPMM_F16) { set_error("y_dtype %d is not a dtype code", y_dtype); return HCSPMM_EINVAL; }
    if (d_in < 1 || d_out < 1 || d_in > (1 << 20) || d_out > (1 << 20)) { set_error("d_in, d_out must be in [1, 2^20]"); return HCSPMM_EINVAL; }
    if (x_dtype != HCSPMM_F32 && x_dtype != HCSPMM_BF16 && x_dtype != HCSPMM_F16) { set_error("x_dtype %d is not a dtype code", x_dtype); return HCSPMM_EINVAL; }
    hcspmm_status st;
    if ((st = check_dense("X", d_X, ldx, d_in)) != HCSPMM_OK) return st;
    if ((st = check_dense("W", d_W, ldw, d_out)) != HCSPMM_OK) return st;
    if ((st = check_dense("Y", d_Y, ldy, d_out)) != HCSPMM_OK) return st;
    const size_t need = hcspmm_aggregate_update_workspace_bytes(plan, d_in, d_out);
    if (!d_workspace || workspace_bytes < need) { set_error("workspace too small: need %zu bytes", need); return HCSPMM_EINVAL; }
    if (((uintptr_t)d_workspace & 255) != 0) { set_error("workspace must be 256-byte aligned"); return HCSPMM_EINVAL; }
    if (plan->n_rows == 0) return HCSPMM_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    float* Z = static_cast<float*>(d_workspace);
    SpmmArgs a{};
    a.n_rows = plan->n_rows; a.n_cols = plan->n_cols; a.rowptr = plan->rowptr; a.colind = plan->colind; a.vals = plan->vals;
    a.X = d_X; a.ldx = ldx; a.d = d_in; a.x_dtype = x_dtype; a.Y = Z; a.ldy = d_in; a.relu = 0;
    // scratch from the shapes alone, for both orders (X W is no wider where it comes first): see hcspmm_gcn_layer_ex
    if ((st = reserve_scratch(const_cast<hcspmm_plan*>(plan), d_in, s)) != HCSPMM_OK) return st;
    if (update_before(plan, a, d_out, y_dtype, need)) {
        HC_HIP(launch_gemm_x(plan->n_cols, d_in, d_out, d_X, ldx, x_dtype, static_cast<const float*>(d_W), ldw, Z, d_out, s));
        a.X = Z; a.ldx = d_out; a.d = d_out; a.x_dtype = HCSPMM_F32;
        a.Y = static_cast<float*>(d_Y); a.ldy = ldy; a.y_dtype = y_dtype; a.relu = apply_relu ? 1 : 0;
        return run_spmm(plan, a, s, nullptr, nullptr, false, nullptr, true);
    }
    return aggregate_then_update(plan, a, static_cast<const float*>(d_W), ldw, d_out, d_Y, ldy, y_dtype, apply_relu, s);
}

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// workspace of the backward pass: S | masked G, or the mask in bits | W^T | partial products of dW
struct BackwardLayout { size_t s_off, gm_off, wt_off, part_off, total; };

static BackwardLayout backward_layout(const hcspmm_plan* plan, int32_t d_in, int32_t d_out)
{
    BackwardLayout l;
    l.s_off = 0;
    l.gm_off = l.s_off + align256((size_t)plan->n_rows * d_out * sizeof(float));
    l.wt_off = l.gm_off + align256((size_t)plan->n_cols * d_out * sizeof(float));
    l.part_off = l.wt_off + align256((size_t)d_in * d_out * sizeof(float));
    l.total = l.part_off + align256((size_t)gemm_tn_spans(plan->n_rows, d_in, d_out) * d_in * d_out * sizeof(float));
    return l;
}

// Whether the backward pass's activation mask rides in the gather, as a bit per element that it looks up beside the rows of G, instead of
// in a masked copy of G, which reads and writes G once more.  Each gathered row costs a request of its own for every 64 columns; rows of a
// window that share columns find their bits in the same lines, scattered ones hardly, so the lines lie by degree and by the windows' distinct
// columns (.70 of the non-zeros and less in communities, .77 and more in power laws).  Whole call, W of 32 columns, copy / bits, us:
//   scattered     169,343 rows of 5, 64 columns: 79 / 71; 1 M of 5, 256: 1780 / 1613, of 8, 128: 1033 / 1021; but of 10: 1146 / 1174,
//                 400,000 of 15, 128: 519 / 544; G of up to 64 MB in whole 128 columns: 100,000 of 10, 128: 104.6 / 98.5, of 21: level;
//                 with columns of padding in the last 64 bits they lose (1 M of 8, 96: 788 / 817)
//   communities   131,072 of 10, 128 columns: 122 / 107, of 23: 145 / 131, 64: 75.2 / 71.8, of 17, 256: 281 / 258; 8,192 of 10, 128: 26.1 / 24.0;
//                 up to 64 columns, where one load asks for a row, not between the L2s of an XCD and of the chip (32,768 of 23, 64:
//                 31.2 / 32.4); 36 and 68 columns lose (131,072 of 35, 36: 85 / 87; 250,048 of 20, 68: 211 / 218, but 132: 442 / 431, 200: 610 / 587)
// What the copy costs falls with G, and a G of a few MB that has just been copied is in the L2s when it is gathered, as the caller's is not; how much then stays of what else
// the call reads goes by X.  From 12 MB of G on (8 where rows are scattered) the bits are ahead whatever X (copy / bits, X of 144 columns: 24,064 rows of 5, 128 columns: 49.9 /
// 48.2, 49,152 in communities of 11, 64: 53.3 / 51.9; but 16,384 of 22, 128: 42.9 / 43.2).  Below they lose behind wide X (4,480 of 10, 128, X of 144: 33.2 / 33.5, of 256: 35.9 /
// 37.4; 8,192 of 8, 128, X of 96: 28.3 / 29.2) and win behind narrow ones from 2 MB on (of 48: 6,016 of 8, 128: 24.4 / 23.1; of up to 128 columns only up to 3 MB: 12,032 in communities
// of 7, 64, X of 128: 24.7 / 23.2, 16,384 of 8: 27.3 / 27.9), at columns of padding not past 6 (16,384 in communities of 16, 132, X of 32: 37.7 / 38.5).  Smaller ones are level or a little
// ahead with some thousand rows and six non-zeros to a row of G (6,016 in communities of 11, 64, X of 48: 18.9 / 18.6, 6,016 of 8: 20.0 / 19.9; but of 5: 19.5 / 20.1,
// 2,112 of 10, 128: 20.4 / 20.7, 4,480 in communities of 11, 96: 19.8 / 20.0).
static bool mask_rides_size(const hcspmm_plan* plan, int32_t d, int32_t d_in, bool shared, double mb)
{
    if (mb >= (shared ? 11.5 : 8.0)) return true;
    if (d_in > 128 || (d % 64 != 0 && mb > 6.0)) return false;
    if (mb >= 2.0) return d_in <= 64 || mb <= 3.0;
    return d_in <= 64 && d % 64 == 0 && plan->n_cols >= 4000 && (shared || plan->nnz >= 6 * (int64_t)plan->n_cols);
}
static bool mask_rides(const hcspmm_plan* plan, const SpmmArgs& a /* with the masked copy for X */, int32_t d_in, const float* G, int64_t ldg, const float* Yf, int64_t ldyf)
{
    if (plan->n_rows == 0 || plan->n_panels > 1 || !(plan->scalar_exec || plan->n_mfma == 0)) return false;
    if (ldg != a.d || (uintptr_t)G % 128 != 0 || !relu_bits_usable(a.d, Yf, ldyf)) return false;     // (rows lie as those of the copy would)
    const bool shared = plan->local || (plan->opt.route_mode != HCSPMM_ROUTE_ALL_CSR && 4 * plan->total_ncols <= 3 * plan->nnz);
    if (a.d % 64 != 0 && (a.d < 96 || !shared)) return false;
    const double mb = (double)plan->n_cols * a.d * 4 / (1 << 20);
    const int64_t most = shared ? (a.d > 64 || mb >= 24.0 ? 30 : 12) : a.d % 128 == 0 && mb <= 64.0 ? 11 : 8;
    return plan->nnz <= most * plan->n_rows && mask_rides_size(plan, a.d, d_in, shared, mb) && csr_mask_usable(a, csr_hints(plan, false));
}

size_t hcspmm_layer_backward_workspace_bytes(const hcspmm_plan* plan, int32_t d_in, int32_t d_out)
{
    if (!plan || d_in < 1 || d_out < 1) return 0;
    return backward_layout(plan, d_in, d_out).total;
}

hcspmm_status hcspmm_layer_backward(const hcspmm_plan* plan, const void* d_G, int64_t ldg, int32_t d_out,
                                    const void* d_Yfwd, int64_t ldyf, const void* d_X, int64_t ldx, int32_t d_in,
                                    const void* d_W, int64_t ldw, void* d_dX, int64_t lddx, void* d_dW, int64_t lddw,
                                    int32_t mask_dx_by_x, void* d_workspace, size_t workspace_bytes, void* stream)
{
    if (!plan) { set_error("plan is NULL"); return HCSPMM_EINVAL; }
    if (d_in < 1 || d_out < 1 || d_in > (1 << 20) || d_out > (1 << 20)) { set_error("d_in, d_out must be in [1, 2^20]"); return HCSPMM_EINVAL; }
    hcspmm_status st;
    if (mask_dx_by_x && d_dX && (st = check_dense("X", d_X, ldx, d_in)) != HCSPMM_OK) return st;
    if ((st = check_dense("G", d_G, ldg, d_out)) != HCSPMM_OK) return st;
    if (d_Yfwd && (st = check_dense("Yfwd", d_Yfwd, ldyf, d_out)) != HCSPMM_OK) return st;
    if ((st = check_dense("W", d_W, ldw, d_out)) != HCSPMM_OK) return st;
    if (d_dX && (st = check_dense("dX", d_dX, lddx, d_in)) != HCSPMM_OK) return st;
    if (d_dW) {
        if ((st = check_dense("dW", d_dW, lddw, d_out)) != HCSPMM_OK) return st;
        if ((st = check_dense("X", d_X, ldx, d_in)) != HCSPMM_OK) return st;
    }
    const BackwardLayout l = backward_layout(plan, d_in, d_out);
    if (!d_workspace || workspace_bytes < l.total) { set_error("workspace too small: need %zu bytes", l.total); return HCSPMM_EINVAL; }
    if (((uintptr_t)d_workspace & 255) != 0) { set_error("workspace must be 256-byte aligned"); return HCSPMM_EINVAL; }
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(d_workspace);
    float* S = reinterpret_cast<float*>(ws + l.s_off);
    float* Gm = reinterpret_cast<float*>(ws + l.gm_off);
    float* Wt = reinterpret_cast<float*>(ws + l.wt_off);
    float* part = reinterpret_cast<float*>(ws + l.part_off);
    const float *G = static_cast<const float*>(d_G), *Yf = static_cast<const float*>(d_Yfwd);
    const bool masked = d_Yfwd && plan->n_cols > 0;
    SpmmArgs a{};
    a.n_rows = plan->n_rows; a.n_cols = plan->n_cols; a.rowptr = plan->rowptr; a.colind = plan->colind; a.vals = plan->vals;
    a.X = masked ? Gm : G; a.ldx = masked ? d_out : ldg; a.d = d_out; a.x_dtype = HCSPMM_F32; a.Y = S; a.ldy = d_out; a.relu = 0;
    // as in hcspmm_aggregate_update; the wave-per-window kernel neither stores S for dW nor applies the mask
    UpdatePlace place = kUpdateApart;
    if (plan->n_rows > 0 && d_dX) {
        place = plan->opt.update_fusion == HCSPMM_UPDATE_FUSED   ? kUpdateEverywhere
                : plan->opt.update_fusion == HCSPMM_UPDATE_SPLIT ? kUpdateApart
                                                                 : update_place(plan, d_out, d_in, HCSPMM_F32, d_dW != nullptr);
        if (place == kUpdateInWindows && (d_dW || mask_dx_by_x)) place = kUpdateApart;
        if (place != kUpdateApart && !update_fusable(a)) place = kUpdateApart;
    }
    if (masked && place == kUpdateApart && mask_rides(plan, a, d_in, G, ldg, Yf, ldyf)) {
        uint2* bits = reinterpret_cast<uint2*>(Gm);             // (8 bytes per row and 64 columns, of 36 columns and more)
        HC_HIP(launch_relu_bits(plan->n_cols, d_out, Yf, ldyf, bits, s));
        a.X = G; a.x_mask = bits;
    } else if (masked) {
        HC_HIP(launch_relu_mask(plan->n_cols, d_out, G, ldg, Yf, ldyf, Gm, d_out, s));
    }
    if (plan->n_rows > 0) {
        if (d_dX) {
            if (place == kUpdateApart && d_dW && !mask_dx_by_x && gemm_grad_usable(plan->n_rows, ldx, d_in, d_out)) {
                if ((st = run_spmm(plan, a, s)) != HCSPMM_OK) return st;
                HC_HIP(launch_gemm_grad(plan->n_rows, static_cast<const float*>(d_X), ldx, d_in, S, d_out, d_out, static_cast<const float*>(d_W), ldw,
                                        static_cast<float*>(d_dX), lddx, static_cast<float*>(d_dW), lddw, part, s));
                return HCSPMM_OK;
            }
            HC_HIP(launch_transpose(d_in, d_out, static_cast<const float*>(d_W), ldw, Wt, s));
            if (place != kUpdateApart) {
                // the next layer's activation mask (its output is this layer's input X) goes into the update's epilogue
                const UpdateArgs u{Wt, d_in, d_in, static_cast<float*>(d_dX), lddx, 0, d_dW ? 1 : 0,
                                   mask_dx_by_x ? static_cast<const float*>(d_X) : nullptr, ldx};
                if ((st = run_spmm(plan, a, s, nullptr, &u, place == kUpdateInWindows)) != HCSPMM_OK) return st;
            } else {
                if ((st = run_spmm(plan, a, s)) != HCSPMM_OK) return st;
                HC_HIP(launch_gemm_f32(plan->n_rows, d_out, d_in, S, d_out, Wt, d_in, static_cast<float*>(d_dX), lddx,
                                       mask_dx_by_x ? static_cast<const float*>(d_X) : nullptr, ldx, s));
            }
        } else if ((st = run_spmm(plan, a, s)) != HCSPMM_OK) {
            return st;
        }
    }
    if (d_dW)
        HC_HIP(launch_gemm_tn(plan->n_rows, static_cast<const float*>(d_X), ldx, d_in, S, d_out, d_out,
                              static_cast<float*>(d_dW), lddw, part, s));
    return HCSPMM_OK;
}

size_t hcspmm_probe_gather_out_bytes(int64_t n, int32_t d)
{
    if (n <= 0 || d < 1) return 256;
    return (size_t)probe_gather_blocks(n, d) * 256 * 4 * sizeof(float);
}

hcspmm_status hcspmm_probe_gather(const int32_t* d_index, int64_t n, const float* d_X, int64_t ldx, int32_t d,
                                  int32_t n_rows_x, float* d_out, size_t out_bytes, void* stream)
{
    if (n < 0 || n_rows_x < 1) { set_error("negative n or empty X"); return HCSPMM_EINVAL; }
    if (d < 4 || d > 256 || d % 4 != 0 || ldx % 4 != 0 || ((uintptr_t)d_X & 15) != 0) {
        set_error("the gather probe needs d a multiple of 4 in [4, 256] and 16-byte aligned X rows");
        return HCSPMM_EUNSUPPORTED;
    }
    hcspmm_status st;
    if ((st = check_dense("X", d_X, ldx, d)) != HCSPMM_OK) return st;
    if (n == 0) return HCSPMM_OK;
    if (!d_index || !d_out) { set_error("NULL argument"); return HCSPMM_EINVAL; }
    if (out_bytes < hcspmm_probe_gather_out_bytes(n, d)) { set_error("out buffer too small: need %zu bytes", hcspmm_probe_gather_out_bytes(n, d)); return HCSPMM_EINVAL; }
    if (((uintptr_t)d_out & 15) != 0) { set_error("out must be 16-byte aligned"); return HCSPMM_EINVAL; }
    HC_HIP(launch_probe_gather(d_index, n, d_X, ldx, d, n_rows_x, d_out, static_cast<hipStream_t>(stream)));
    return HCSPMM_OK;
}

hcspmm_status hcspmm_plan_set_update_fusion(hcspmm_plan* plan, int32_t update_fusion)
{
    if (!plan) { set_error("plan is NULL"); return HCSPMM_EINVAL; }
    if (update_fusion < 0 || update_fusion > 2) { set_error("bad update_fusion"); return HCSPMM_EINVAL; }
    plan->opt.update_fusion = update_fusion;
    return HCSPMM_OK;
}

void hcspmm_plan_destroy(hcspmm_plan* plan)
{
    if (!plan) return;
    (void)hipDeviceSynchronize();
    if (plan->side[0]) (void)hipStreamDestroy(plan->side[0]);
    if (plan->side[1]) (void)hipStreamDestroy(plan->side[1]);
    if (plan->ev_fork) (void)hipEventDestroy(plan->ev_fork);
    if (plan->ev_join[0]) (void)hipEventDestroy(plan->ev_join[0]);
    if (plan->ev_join[1]) (void)hipEventDestroy(plan->ev_join[1]);
    free_plan_arrays(plan);
    if (plan->cache) { plan->cache->clear(); delete plan->cache; }
    delete plan;
}

const char* hcspmm_status_string(hcspmm_status s)
{
    switch (s) {
        case HCSPMM_OK: return "ok";
        case HCSPMM_EINVAL: return "invalid argument";
        case HCSPMM_EBADCSR: return "invalid CSR";
        case HCSPMM_EALLOC: return "allocation failed";
        case HCSPMM_EHIP: return "HIP runtime error";
        case HCSPMM_EUNSUPPORTED: return "unsupported";
    }
    return "unknown status";
}

const char* hcspmm_last_error(void) { return g_err; }

int32_t hcspmm_version(void) { return 10100; }

}  // extern "C"
