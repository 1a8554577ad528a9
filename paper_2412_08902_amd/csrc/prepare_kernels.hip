// Preprocessing kernels: row windows, condensing, window features, selection, launch tables.
//
// Section IV-A: A is cut into windows of 16 rows and each window's non-zero columns are moved to
// the front.  Here "moved to the front" is materialised as (a) the ascending list of the
// window's distinct column ids and (b) for every non-zero the position of its column in that
// list.  Section IV-C: the per-window features (number of non-zero columns, sparsity) feed a
// three-parameter linear model whose sign picks the path; it is evaluated in exact integers.
#include <algorithm>

#include "common.hpp"

namespace hcspmm {

// ------------------------------------------------------------------------------------------------
// block-wide exclusive scan of one int per thread (NT threads, NT a multiple of 64, NT <= 1024)
// ------------------------------------------------------------------------------------------------
template <int NT>
__device__ inline int block_exclusive_scan(int v, int* total, int* smem /* NT/64 + 1 ints */)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int t = __shfl_up(inc, off, 64);
        if (lane >= off) inc += t;
    }
    __syncthreads();                       // smem may still be in use by a previous call
    if (lane == 63) smem[wave] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int i = 0; i < NT / 64; ++i) { int t = smem[i]; smem[i] = run; run += t; }
        smem[NT / 64] = run;
    }
    __syncthreads();
    *total = smem[NT / 64];
    return smem[wave] + inc - v;
}

// ------------------------------------------------------------------------------------------------
// generic device-wide exclusive scan  int32[n] -> int64[n+1]
// ------------------------------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

size_t scan_scratch_elems(int64_t n) { return (size_t)((n + kScanTile - 1) / kScanTile) + 2; }

__global__ __launch_bounds__(kScanThreads) void k_scan_tile_sums(const int32_t* __restrict__ in, int64_t n,
                                                                 int64_t* __restrict__ tile_sums)
{
    __shared__ long long part[kScanThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    long long acc = 0;
    for (int i = 0; i < kScanItems; ++i) {
        int64_t idx = base + (int64_t)i * kScanThreads + threadIdx.x;
        if (idx < n) acc += in[idx];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int i = 0; i < kScanThreads / 64; ++i) t += part[i];
        tile_sums[blockIdx.x] = t;
    }
}

// one workgroup walks the tile sums in order (there are at most a few hundred thousand)
__global__ __launch_bounds__(256) void k_scan_tile_offsets(int64_t* __restrict__ tile_sums, int64_t n_tiles)
{
    __shared__ long long wsum[4];
    __shared__ long long carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    for (int64_t base = 0; base < n_tiles; base += 256) {
        int64_t idx = base + threadIdx.x;
        long long v = idx < n_tiles ? tile_sums[idx] : 0;
        long long inc = v;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            long long t = __shfl_up(inc, off, 64);
            if (lane >= off) inc += t;
        }
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        long long wave_off = 0;
        for (int i = 0; i < wave; ++i) wave_off += wsum[i];
        long long carry = carry_s;
        if (idx < n_tiles) tile_sums[idx] = carry + wave_off + inc - v;
        __syncthreads();
        if (threadIdx.x == 255) carry_s = carry + wave_off + inc;
        __syncthreads();
    }
    if (threadIdx.x == 0) tile_sums[n_tiles] = carry_s;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const int32_t* __restrict__ in, int64_t n,
                                                             const int64_t* __restrict__ tile_offsets,
                                                             int64_t n_tiles, int64_t* __restrict__ out)
{
    __shared__ int smem[kScanThreads / 64 + 1];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int v[kScanItems];
    int local = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        int64_t idx = base + i;
        v[i] = idx < n ? in[idx] : 0;
        local += v[i];
    }
    int total;
    // int suffices inside one tile: every array scanned here sums to less than 2^31 overall
    long long off = (long long)block_exclusive_scan<kScanThreads>(local, &total, smem);
    long long run = tile_offsets[blockIdx.x] + off;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        int64_t idx = base + i;
        if (idx < n) out[idx] = run;
        run += v[i];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = tile_offsets[n_tiles];
}

hipError_t exclusive_scan_i32_i64(const int32_t* in, int64_t n, int64_t* out, int64_t* scratch, hipStream_t stream)
{
    if (n <= 0) return hipMemsetAsync(out, 0, sizeof(int64_t), stream);
    const int64_t n_tiles = (n + kScanTile - 1) / kScanTile;
    hipLaunchKernelGGL(k_scan_tile_sums, dim3((unsigned)n_tiles), dim3(kScanThreads), 0, stream, in, n, scratch);
    hipLaunchKernelGGL(k_scan_tile_offsets, dim3(1), dim3(256), 0, stream, scratch, n_tiles);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)n_tiles), dim3(kScanThreads), 0, stream, in, n, scratch, n_tiles,
                       out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// several arrays of one length scanned by one three-kernel sequence (the preprocessing is bound by
// the number of its small launches and read-backs, not by their work)
// ------------------------------------------------------------------------------------------------
size_t scan_multi_scratch_elems(int64_t n) { return (size_t)kScanMaxArrays * scan_scratch_elems(n); }

__global__ __launch_bounds__(kScanThreads) void k_scan_tile_sums_m(ScanMulti m, int64_t n, int64_t stride,
                                                                   int64_t* __restrict__ tile_sums)
{
    __shared__ long long part[kScanThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    for (int a = 0; a < m.k; ++a) {
        const int32_t* __restrict__ in = m.in[a];
        long long acc = 0;
        for (int i = 0; i < kScanItems; ++i) {
            const int64_t idx = base + (int64_t)i * kScanThreads + threadIdx.x;
            if (idx < n) acc += in[idx];
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
        __syncthreads();                                        // part[] of the previous array has been read
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            long long t = 0;
            for (int i = 0; i < kScanThreads / 64; ++i) t += part[i];
            tile_sums[a * stride + blockIdx.x] = t;
        }
    }
}

// workgroup a walks the tile sums of array a in order; totals[a] receives the array's sum
__global__ __launch_bounds__(256) void k_scan_tile_offsets_m(int64_t* __restrict__ tile_sums_all, int64_t n_tiles,
                                                             int64_t stride, int64_t* __restrict__ totals)
{
    __shared__ long long wsum[4];
    __shared__ long long carry_s;
    int64_t* __restrict__ tile_sums = tile_sums_all + blockIdx.x * stride;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    for (int64_t base = 0; base < n_tiles; base += 256) {
        const int64_t idx = base + threadIdx.x;
        const long long v = idx < n_tiles ? tile_sums[idx] : 0;
        long long inc = v;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const long long t = __shfl_up(inc, off, 64);
            if (lane >= off) inc += t;
        }
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        long long wave_off = 0;
        for (int i = 0; i < wave; ++i) wave_off += wsum[i];
        const long long carry = carry_s;
        if (idx < n_tiles) tile_sums[idx] = carry + wave_off + inc - v;
        __syncthreads();
        if (threadIdx.x == 255) carry_s = carry + wave_off + inc;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        tile_sums[n_tiles] = carry_s;
        if (totals) totals[blockIdx.x] = carry_s;
    }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply_m(ScanMulti m, int64_t n, int64_t stride,
                                                               const int64_t* __restrict__ tile_offsets_all,
                                                               int64_t n_tiles)
{
    __shared__ int smem[kScanThreads / 64 + 1];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    for (int a = 0; a < m.k; ++a) {
        int64_t* __restrict__ out = m.out[a];
        if (!out) continue;                                     // only the total of this array was wanted
        const int32_t* __restrict__ in = m.in[a];
        const int64_t* __restrict__ tile_offsets = tile_offsets_all + a * stride;
        int v[kScanItems];
        int local = 0;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) {
            const int64_t idx = base + i;
            v[i] = idx < n ? in[idx] : 0;
            local += v[i];
        }
        int total;
        const long long off = (long long)block_exclusive_scan<kScanThreads>(local, &total, smem);
        long long run = tile_offsets[blockIdx.x] + off;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) {
            const int64_t idx = base + i;
            if (idx < n) out[idx] = run;
            run += v[i];
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = tile_offsets[n_tiles];
    }
}

hipError_t exclusive_scan_multi(const ScanMulti& m, int64_t n, int64_t* totals_dev, int64_t* scratch, hipStream_t stream)
{
    if (m.k < 1 || m.k > kScanMaxArrays) return hipErrorInvalidValue;
    if (n <= 0) {
        for (int a = 0; a < m.k; ++a)
            if (m.out[a]) { hipError_t e = hipMemsetAsync(m.out[a], 0, sizeof(int64_t), stream); if (e != hipSuccess) return e; }
        if (totals_dev) return hipMemsetAsync(totals_dev, 0, (size_t)m.k * sizeof(int64_t), stream);
        return hipSuccess;
    }
    const int64_t n_tiles = (n + kScanTile - 1) / kScanTile;
    const int64_t stride = (int64_t)scan_scratch_elems(n);
    hipLaunchKernelGGL(k_scan_tile_sums_m, dim3((unsigned)n_tiles), dim3(kScanThreads), 0, stream, m, n, stride, scratch);
    hipLaunchKernelGGL(k_scan_tile_offsets_m, dim3((unsigned)m.k), dim3(256), 0, stream, scratch, n_tiles, stride, totals_dev);
    hipLaunchKernelGGL(k_scan_apply_m, dim3((unsigned)n_tiles), dim3(kScanThreads), 0, stream, m, n, stride, scratch, n_tiles);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// per-window non-zero count, and the list of windows too large for the LDS sort
// ------------------------------------------------------------------------------------------------
__device__ inline void window_span(int32_t w, int32_t n_rows, const int32_t* __restrict__ rowptr, int32_t& s,
                                   int32_t& e)
{
    int64_t r0 = (int64_t)w * kH;
    int64_t r1 = r0 + kH;
    if (r1 > n_rows) r1 = n_rows;
    s = rowptr[r0];
    e = rowptr[r1];
}

__global__ __launch_bounds__(256) void k_window_nnz(int32_t W, int32_t n_rows, const int32_t* __restrict__ rowptr,
                                                    int32_t* __restrict__ nnzw, int32_t* __restrict__ big_list,
                                                    int32_t* __restrict__ big_count)
{
    int32_t w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= W) return;
    int32_t s, e;
    window_span(w, n_rows, rowptr, s, e);
    nnzw[w] = e - s;
    if (e - s > kUniqueSmallCap) big_list[atomicAdd(big_count, 1)] = w;
}

hipError_t launch_window_nnz(int32_t W, int32_t n_rows, const int32_t* rowptr, int32_t* nnzw, int32_t* big_list,
                             int32_t* big_count, hipStream_t s)
{
    hipLaunchKernelGGL(k_window_nnz, dim3((W + 255) / 256), dim3(256), 0, s, W, n_rows, rowptr, nnzw, big_list,
                       big_count);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// condensing, small windows: sort the window's column ids in LDS, keep the distinct ones
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_unique_small(int32_t W, int32_t n_rows, const int32_t* __restrict__ rowptr,
                                                      const int32_t* __restrict__ colind,
                                                      int32_t* __restrict__ tmp_cols, int32_t* __restrict__ ncols,
                                                      const uint8_t* __restrict__ route /* may be null: every window */)
{
    __shared__ int32_t keys[kUniqueSmallCap];
    __shared__ int smem[256 / 64 + 1];
    const int32_t w = blockIdx.x;
    if (route && route[w] == 0) return;          // only the matrix path's windows need the list
    int32_t s, e;
    window_span(w, n_rows, rowptr, s, e);
    const int32_t n = e - s;
    if (n > kUniqueSmallCap) return;             // handled by k_unique_big
    if (n == 0) {
        if (threadIdx.x == 0) ncols[w] = 0;
        return;
    }
    int P = 2;
    while (P < n) P <<= 1;
    for (int i = threadIdx.x; i < P; i += 256) keys[i] = i < n ? colind[s + i] : 0x7fffffff;
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < (P >> 1); t += 256) {
                int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                int p = i | j;
                bool up = (i & k) == 0;
                int32_t a = keys[i], b = keys[p];
                if ((a > b) == up) { keys[i] = b; keys[p] = a; }
            }
            __syncthreads();
        }
    }
    // distinct values: thread t owns the contiguous slice [t*ipt, (t+1)*ipt)
    const int ipt = (P + 255) / 256;
    const int lo = threadIdx.x * ipt;
    int cnt = 0;
    for (int i = lo; i < lo + ipt && i < n; ++i) cnt += (i == 0 || keys[i] != keys[i - 1]) ? 1 : 0;
    int total;
    int off = block_exclusive_scan<256>(cnt, &total, smem);
    for (int i = lo; i < lo + ipt && i < n; ++i)
        if (i == 0 || keys[i] != keys[i - 1]) tmp_cols[(int64_t)s + off++] = keys[i];
    if (threadIdx.x == 0) ncols[w] = total;
}

hipError_t launch_unique_small(int32_t W, int32_t n_rows, const int32_t* rowptr, const int32_t* colind,
                               int32_t* tmp_cols, int32_t* ncols, const uint8_t* route, hipStream_t s)
{
    hipLaunchKernelGGL(k_unique_small, dim3(W), dim3(256), 0, s, W, n_rows, rowptr, colind, tmp_cols, ncols, route);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// condensing, large windows: an LDS bitmap over a range of 2^20 columns per pass
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_unique_big(const int32_t* __restrict__ big_list, int32_t n_rows,
                                                     int32_t n_cols, const int32_t* __restrict__ rowptr,
                                                     const int32_t* __restrict__ colind,
                                                     int32_t* __restrict__ tmp_cols, int32_t* __restrict__ ncols,
                                                     const uint8_t* __restrict__ route /* may be null: every listed window */)
{
    __shared__ uint32_t bm[kBitmapWords];
    __shared__ int smem[1024 / 64 + 1];
    constexpr int kBits = kBitmapWords * 32;
    constexpr int kWordsPerThread = kBitmapWords / 1024;
    const int32_t w = big_list[blockIdx.x];
    if (route && route[w] == 0) return;
    int32_t s, e;
    window_span(w, n_rows, rowptr, s, e);
    int32_t running = 0;
    for (int64_t base = 0; base < n_cols; base += kBits) {
        for (int i = threadIdx.x; i < kBitmapWords; i += 1024) bm[i] = 0u;
        __syncthreads();
        for (int32_t k = s + threadIdx.x; k < e; k += 1024) {
            int64_t c = (int64_t)colind[k] - base;
            if (c >= 0 && c < kBits) atomicOr(&bm[c >> 5], 1u << (c & 31));
        }
        __syncthreads();
        const int w0 = threadIdx.x * kWordsPerThread;
        int cnt = 0;
#pragma unroll 4
        for (int i = 0; i < kWordsPerThread; ++i) cnt += __popc(bm[w0 + i]);
        int total;
        int off = block_exclusive_scan<1024>(cnt, &total, smem);
        int32_t* out = tmp_cols + (int64_t)s + running + off;
        for (int i = 0; i < kWordsPerThread; ++i) {
            uint32_t bits = bm[w0 + i];
            while (bits) {
                int b = __ffs(bits) - 1;
                bits &= bits - 1;
                *out++ = (int32_t)(base + (int64_t)(w0 + i) * 32 + b);
            }
        }
        running += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) ncols[w] = running;
}

hipError_t launch_unique_big(int32_t n_big, const int32_t* big_list, int32_t n_rows, int32_t n_cols,
                             const int32_t* rowptr, const int32_t* colind, int32_t* tmp_cols, int32_t* ncols,
                             const uint8_t* route, hipStream_t s)
{
    if (n_big <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_unique_big, dim3(n_big), dim3(1024), 0, s, big_list, n_rows, n_cols, rowptr, colind, tmp_cols,
                       ncols, route);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// From the CSR arrays to a plan's launch tables in three to seven launches and one read-back.
//
// A preparation's work is small (a medium graph: ~40 us of kernels), so launches and synchronisations are what it costs.
// (27 launches, three-kernel scans over arrays of flags and six read-backs took 240 us on 17,000 rows and 490 us on
// 169,000, most of it in the scans' few wavefronts and in waiting.)  Here every kernel leaves at once when an earlier one
// has found the CSR arrays unsound, so nothing waits for the host in between; flags are recomputed from the row offsets
// where they are needed instead of being written, scanned and read back; and a tile of 64 windows (1024 rows) writes its
// sums once, from which every workgroup of the next kernel adds up its own offset (2,400 tiles, those of 2.4 M rows, are
// 153 KB of window sums out of L2 per workgroup).  That grows with the square of the rows, so matrices of more than
// kDirectTiles tiles also get sums per group of 256 tiles (k_group_sums, a launch more per array of sums), and a workgroup
// adds up groups and the tiles of its own group: 1.02 G rows are 1 M tiles and 3,900 groups.  The totals go straight into a
// page of host memory.
//   k_pre_validate   row offsets; non-zeros per window; windows by size class
//   k_pre_count*     distinct columns per window by LDS hash sets (bitmap passes beyond their capacity), range of the columns;
//                    one launch for few windows (and no k_pre_validate, if they are all, nor k_pre_select), one per size class for many
//   k_pre_sorted, k_pre_sample   where they decide something: whether rows ascend, how much neighbouring rows share
//   k_pre_select     selection per window, sums per tile
//   k_pre_rows       launch guard, route and list offset per window, row classes, sums per tile
//   k_pre_fill       row lists, segments of long rows, totals
// ------------------------------------------------------------------------------------------------
constexpr int kTileWindows = 64, kTileRows = kTileWindows * kH;
constexpr int kBigTakes1kWindows = 16384;
constexpr int kWt = 8, kRt = 4;                                 // 64-bit sums per tile: windows, rows
constexpr int kGroupTiles = 256, kDirectTiles = 4096;

static int32_t group_count(int32_t n_tiles) { return n_tiles > kDirectTiles ? (n_tiles + kGroupTiles - 1) / kGroupTiles : 0; }
size_t prep_tile_count(int32_t W) { return (size_t)((W + kTileWindows - 1) / kTileWindows > 0 ? (W + kTileWindows - 1) / kTileWindows : 1); }
size_t prep_tile_words(int32_t W) { const size_t n = prep_tile_count(W); return (n + (size_t)group_count((int32_t)n)) * (kWt + kRt); }
void prep_bind_sums(Prep& p, unsigned long long* words)
{
    p.n_tiles = (int32_t)prep_tile_count(p.W);
    const int32_t groups = group_count(p.n_tiles);
    p.wt = words;
    p.rt = p.wt + (size_t)kWt * p.n_tiles;
    p.wg = groups ? p.rt + (size_t)kRt * p.n_tiles : nullptr;
    p.rg = groups ? p.wg + (size_t)kWt * groups : nullptr;
}
size_t panel_sum_words(int32_t n_panels, int32_t n_tiles) { return 3 * (size_t)n_panels * ((size_t)n_tiles + (size_t)group_count(n_tiles)); }

template <class T> __device__ inline T wave_sum(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Inclusive prefixes over a wave by DPP moves (a 64-bit shuffle is two trips through LDS, six in a row for a sum).
template <int CTRL, int ROWS> __device__ __forceinline__ unsigned long long dpp_u64(unsigned long long v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xf, false);
    return (unsigned long long)hi << 32 | lo;
}
__device__ __forceinline__ unsigned long long wave_scan_u64(unsigned long long v)
{
    v += dpp_u64<0x111, 0xf>(v);                                // row_shr 1, 2, 4, 8
    v += dpp_u64<0x112, 0xf>(v);
    v += dpp_u64<0x114, 0xf>(v);
    v += dpp_u64<0x118, 0xf>(v);
    v += dpp_u64<0x142, 0xa>(v);                                // row_bcast 15, 31
    v += dpp_u64<0x143, 0xc>(v);
    return v;
}
__device__ __forceinline__ unsigned long long lane_u64(unsigned long long v, int lane)
{
    return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) { return lane_u64(wave_scan_u64(v), 63); }

// sums of several values over the workgroup's 256 threads, in every thread: two barriers for all of them
template <int N> __device__ inline void block_sums_u64(unsigned long long (&v)[N], unsigned long long* smem /* 4 * N */)
{
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = wave_sum_u64(v[i]);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int i = 0; i < N; ++i) smem[(threadIdx.x >> 6) * N + i] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = smem[i] + smem[N + i] + smem[2 * N + i] + smem[3 * N + i];
}
__device__ inline unsigned long long block_sum_u64(unsigned long long v, unsigned long long* smem /* 4 */)
{
    unsigned long long one[1] = {v};
    block_sums_u64<1>(one, smem);
    return one[0];
}

// exclusive prefixes of several values over the workgroup's 256 threads
template <int N> __device__ inline void block_scans_u64(unsigned long long (&v)[N], unsigned long long* smem /* 4 * N */)
{
    const int wave = threadIdx.x >> 6;
    unsigned long long inc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) inc[i] = wave_scan_u64(v[i]);
    __syncthreads();
    if ((threadIdx.x & 63) == 63)
#pragma unroll
        for (int i = 0; i < N; ++i) smem[wave * N + i] = inc[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i)
        v[i] = (wave > 0 ? smem[i] : 0ull) + (wave > 1 ? smem[N + i] : 0ull) + (wave > 2 ? smem[2 * N + i] : 0ull) + inc[i] - v[i];
}
__device__ inline unsigned long long block_scan_u64(unsigned long long v, unsigned long long* smem /* 4 */)
{
    unsigned long long one[1] = {v};
    block_scans_u64<1>(one, smem);
    return one[0];
}

// sums of 256 tiles each (K values per tile); blockIdx.y: one array of tiles after the other
template <int K>
__global__ __launch_bounds__(256) void k_group_sums(int32_t n_tiles, const unsigned long long* __restrict__ tiles, unsigned long long* __restrict__ groups)
{
    __shared__ unsigned long long smem[4 * K];
    const int t = blockIdx.x * kGroupTiles + threadIdx.x;
    const unsigned long long* __restrict__ in = tiles + ((int64_t)blockIdx.y * n_tiles + t) * K;
    unsigned long long v[K];
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] = t < n_tiles ? in[i] : 0ull;
    block_sums_u64<K>(v, smem);
    if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < K; ++i) groups[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * K + i] = v[i];
}

// Calls f(sums, in front of tile `at`) for tiles, or groups of tiles, that make up all tiles together (ALL) or those in
// front of `at`; the callers `thread` of `threads` share them.  groups: null where there are no group sums.
template <int K, bool ALL, class F>
__device__ __forceinline__ void for_sums(const unsigned long long* __restrict__ tiles, const unsigned long long* __restrict__ groups, int n_tiles,
                                         int at, int thread, int threads, F&& f)
{
    int first = 0, last = ALL ? n_tiles : at;
    if (groups) {
        const int own = at / kGroupTiles, n = ALL ? (n_tiles + kGroupTiles - 1) / kGroupTiles : own;
        for (int g = thread; g < n; g += threads)
            if (g != own) f(groups + (int64_t)g * K, g < own);
        first = own * kGroupTiles;
        last = min(last, first + kGroupTiles);
    }
    for (int t = first + thread; t < last; t += threads) f(tiles + (int64_t)t * K, t < at);
}

// selection (Section IV-C): z' = c0*H*ncols^2 + c1*(H*ncols - nnzw) + c2*H*ncols ; matrix path iff z' < 0
__device__ inline int window_route(const Prep& p, int mode, long long nc, long long nz)
{
    if (nc <= 0 || mode == HCSPMM_ROUTE_ALL_CSR) return 0;
    if (mode == HCSPMM_ROUTE_ALL_MFMA) return 1;
    // |c*| < 2^40 and H*ncols^2 < 2^58: every factor fits 64 bits, and 128-bit sums of their products keep the sign exact
    const long long hn = (long long)kH * nc;
    const __int128 z = (__int128)p.c0 * (hn * nc) + (__int128)p.c1 * (hn - nz) + (__int128)p.c2 * hn;
    return z < 0 ? 1 : 0;
}

// windows on the matrix path | ... of the wave-per-window kernel | medium | wide, 16 bits each (a tile has 64 windows, a
// group of tiles 16,384)
__device__ inline unsigned long long window_counts(int r, long long nc)
{
    if (!r) return 0ull;
    return 1ull | (nc <= kMfmaSmallMaxCols ? 1ull << 16 : nc <= kMfmaMidMaxCols ? 1ull << 32 : 1ull << 48);
}

// What a window adds to its tile's sums: [0] distinct columns; [1] non-zeros, [2] window counts, [3] columns of wide windows on the matrix path under
// the plan's own mode, [7] columns there; [4..6] as [1..3] with every window there (what the launch guard may decide for)
__device__ inline void window_sums(int route /* under the plan's own mode */, long long nc, long long nz, unsigned long long (&v)[kWt])
{
    v[0] = (unsigned long long)nc;
    v[7] = 0ull;
#pragma unroll
    for (int set = 0; set < 2; ++set) {
        const int r = set == 0 ? route : nc > 0;
        v[1 + 3 * set] = r ? (unsigned long long)nz : 0ull;
        v[2 + 3 * set] = window_counts(r, nc);
        v[3 + 3 * set] = r && nc > kMfmaMidMaxCols ? (unsigned long long)nc : 0ull;
        if (set == 0 && r) v[7] = (unsigned long long)nc;
    }
}
// ... added by one thread (whole numbers: in any order, and what is taken off again leaves no trace)
__device__ inline void add_to_tile(const Prep& p, int32_t w, const unsigned long long (&v)[kWt], bool off = false)
{
    unsigned long long* __restrict__ to = p.wt + (int64_t)(w / kTileWindows) * kWt;
#pragma unroll
    for (int i = 0; i < kWt; ++i)
        if (v[i]) atomicAdd(to + i, off ? 0ull - v[i] : v[i]);
}

// The size class of a window of n non-zeros: on the lists of the larger ones, and of those that k_pre_count_1k counts.
__device__ inline void list_window(const Prep& p, int32_t w, int32_t n, bool count_1k)
{
    if (n > kCountMidCap) p.huge_list[atomicAdd(p.ctl + 2, 1)] = w;
    else if (n > kUniqueSmallCap) p.big_list[atomicAdd(p.ctl + 1, 1)] = w;
    else if (n > kCountTinyCap && count_1k) p.count_1k[atomicAdd(p.ctl + 3, 1)] = w;
}

// SUMS: the tiles' sums of windows are added up here, with the counts carried over, and k_pre_count_few puts the touched windows right
template <bool SUMS>
__global__ __launch_bounds__(256) void k_pre_validate(Prep p)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i == 0) {
        if (p.rowptr[0] != 0) atomicOr(p.ctl, 1);
        if ((int64_t)p.rowptr[p.n_rows] != p.nnz) atomicOr(p.ctl, 2);
    }
    if (!SUMS && i >= p.n_rows) return;
    const int64_t r = min(i, (int64_t)p.n_rows - 1);
    const int32_t a = p.rowptr[r], b = p.rowptr[r + 1];
    if (a < 0 || b < a) atomicOr(p.ctl, 4);
    const bool first = i % kH == 0 && i < p.n_rows;             // of a window
    if (!SUMS && !first) return;
    // (differences of unsound offsets are only ever compared; nothing indexes with them)
    const int32_t w = (int32_t)(r / kH);
    unsigned long long v[kWt] = {};
    if (first) {
        const int32_t n = p.rowptr[min(i + kH, (int64_t)p.n_rows)] - a, nc = p.old_ncols ? p.old_ncols[w] : 0;
        p.nnzw[w] = n;
        if (p.old_ncols || !p.features) p.ncols[w] = nc;        // counts of untouched windows are carried over; a scalar-only plan counts on first request
        if (p.features) list_window(p, w, n, !p.touched);
        if constexpr (SUMS) window_sums(window_route(p, p.mode, nc, n), nc, n, v);
    }
    if constexpr (SUMS) {                                       // (a wave's four windows are of one tile)
#pragma unroll
        for (int j = 0; j < kWt; ++j) {
            v[j] += __shfl_xor(v[j], 16, 64);
            v[j] += __shfl_xor(v[j], 32, 64);
        }
        if ((threadIdx.x & 63) == 0) add_to_tile(p, w, v);
    }
}

// Distinct columns of kSamples stretches of p.sample_len consecutive non-zeros, spread over the matrix, added up in ctl[8]: how
// many X rows the rows that run side by side share (windows of 16 rows say nothing of that: a community of a few thousand
// nodes is as scattered inside a window as a power-law graph).  One bit per column of a set of 32 * WORDS bits, eight times
// the stretch; columns that share a bit hide some six in a hundred distinct ones at most.
constexpr int kSamples = 64;
template <int NT, int WORDS>
__device__ inline void sample_stretch(const Prep& p, int s, uint32_t* bm /* WORDS + 1 */)
{
    const int64_t k0 = (p.nnz - p.sample_len) * s / (kSamples - 1);
    for (int i = threadIdx.x; i <= WORDS; i += NT) bm[i] = 0u;
    __syncthreads();
    constexpr int AHEAD = 16;
    for (int i = threadIdx.x; i < p.sample_len; i += NT * AHEAD) {
        uint32_t c[AHEAD];
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) c[j] = (uint32_t)p.colind[k0 + min(i + NT * j, p.sample_len - 1)];
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            const uint32_t bit = (c[j] ^ (c[j] / (WORDS * 32)) * 0x9E375u) % (WORDS * 32);
            atomicOr(&bm[bit >> 5], 1u << (bit & 31));
        }
    }
    __syncthreads();
    uint32_t n = 0;
    for (int i = threadIdx.x; i < WORDS; i += NT) n += __popc(bm[i]);
    atomicAdd(&bm[WORDS], n);
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(p.ctl + 8, (int)bm[WORDS]);
}
__global__ __launch_bounds__(1024) void k_pre_sample(Prep p)
{
    __shared__ uint32_t bm[kSamplePanels * 8 / 32 + 1];
    if (*p.ctl & 7) return;
    sample_stretch<1024, kSamplePanels * 8 / 32>(p, blockIdx.x, bm);
}
double sample_share(const Prep& p, int32_t distinct) { return p.sample_len > 0 ? (double)distinct / ((double)kSamples * p.sample_len) : 1.0; }

// columns only (a plan that counts nothing still checks them); the first kSamples workgroups take the short sample, if any
__global__ __launch_bounds__(256) void k_validate_cols(Prep p, int samples)
{
    __shared__ uint32_t bm[kSampleSlices * 8 / 32 + 1];
    if ((int)blockIdx.x < samples) {
        sample_stretch<256, kSampleSlices * 8 / 32>(p, blockIdx.x, bm);
        return;
    }
    const int64_t stride = (int64_t)(gridDim.x - samples) * 256;
    bool bad = false;
    for (int64_t k = (int64_t)(blockIdx.x - samples) * 256 + threadIdx.x; k < p.nnz; k += stride) {
        const int32_t c = p.colind[k];
        bad |= (c < 0 || c >= p.n_cols);
    }
    if (bad) atomicOr(p.ctl, 8);
}

// rows whose columns do not ascend (a descent inside a row; descents at row starts are looked up)
__global__ __launch_bounds__(256) void k_pre_sorted(Prep p)
{
    if (*p.ctl & 7) return;
    const int64_t stride = (int64_t)gridDim.x * 256;
    bool bad = false;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x + 1; k < p.nnz; k += stride) {
        if (p.colind[k - 1] <= p.colind[k]) continue;
        int32_t lo = 0, hi = p.n_rows;                          // first row that starts at or behind k
        while (lo < hi) { const int32_t mid = lo + ((hi - lo) >> 1); if (p.rowptr[mid] < k) lo = mid + 1; else hi = mid; }
        bad |= p.rowptr[lo] != k;
    }
    if (bad) atomicOr(p.ctl + 6, 1);
}

// Inserts the column ids of non-zeros s .. e-1 into an open-addressing set of at least twice as many entries (linear probing, empty = -1; an id
// outside the matrix is reported and left out) and returns how many insertions found an empty slot.  The set is never more
// than half full, so every probe sequence ends.  nt threads count one window (tid: the caller's place among them); several
// such groups of a workgroup may each count their own, one that has none calls with s = e (the barriers are the
// workgroup's).
__device__ inline int count_distinct(int32_t s, int32_t e, const Prep& p, int32_t* table, int* smem /* nt / 64 */, int tid, int nt)
{
    const int32_t n = e - s;
    int T = nt;                                   // power of two, at least twice the entries
    while (T < 2 * n) T <<= 1;
    const uint32_t mask = (uint32_t)T - 1;
    if (n > 0)
#pragma unroll 1
        for (int i = tid; i < T; i += nt) table[i] = -1;
    __syncthreads();
    int cnt = 0;
    bool bad = false;
    for (int32_t k0 = s + tid; k0 < e; k0 += 4 * nt) {          // (four loads in flight: a window is little else than their latency)
        int32_t col[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) col[j] = p.colind[min(k0 + j * nt, e - 1)];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (k0 + j * nt >= e) break;
            const int32_t c = col[j];
            if (c < 0 || c >= p.n_cols) { bad = true; continue; }
            uint32_t h = ((uint32_t)c * 0x9E3779B1u >> 12) & mask;
            for (;;) {
                const int32_t prev = atomicCAS(&table[h], -1, c);
                if (prev == -1) { ++cnt; break; }
                if (prev == c) break;
                h = (h + 1) & mask;
            }
        }
    }
    if (bad) atomicOr(p.ctl, 8);
    cnt = wave_sum(cnt);
    if ((tid & 63) == 0) smem[tid >> 6] = cnt;
    __syncthreads();
    int total = 0;
#pragma unroll 1
    for (int i = 0; i < nt / 64; ++i) total += smem[i];
    return total;
}

// The same for a window of any size by the NT threads of the workgroup, with a bitmap of 32 * `words` columns a pass.  A thread takes four entries in a
// row, eight times that requested together (one after the other a window of 21,000 non-zeros is 21 trips to memory for 1024 threads), and
// sets the bits of one word at once: neighbouring entries of a row mostly share words, and lanes that add to the same word take turns.
// (Hubs of 154,000 non-zeros to a window: the launch 44 -> 20 us.)
typedef int32_t i4_any __attribute__((ext_vector_type(4), aligned(4)));
template <int NT>
__device__ inline int count_bits(int32_t s, int32_t e /* at least s + 4 */, const Prep& p, uint32_t* __restrict__ bm, int words, int* smem /* NT / 64 */)
{
    constexpr uint32_t U = 8;
    const uint32_t bits_a_pass = (uint32_t)words * 32u;
    int cnt = 0;
    bool bad = false;
    for (int64_t base = 0; base < p.n_cols; base += bits_a_pass) {
#pragma unroll 1
        for (int j = threadIdx.x; j < words; j += NT) bm[j] = 0u;
        __syncthreads();
        for (uint32_t k0 = (uint32_t)s + 4 * threadIdx.x; k0 < (uint32_t)e; k0 += 4 * NT * U) {
            i4_any col[U];
#pragma unroll
            for (uint32_t j = 0; j < U; ++j)                    // (the last four entries instead of what lies behind them)
                col[j] = *reinterpret_cast<const i4_any*>(p.colind + min(k0 + j * 4 * NT, (uint32_t)e - 4u));
#pragma unroll
            for (uint32_t j = 0; j < U; ++j) {
                if (k0 + j * 4 * NT >= (uint32_t)e) break;
                uint32_t at = ~0u, bits = 0u;                   // word, and bits to set in it
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if ((uint32_t)col[j][i] >= (uint32_t)p.n_cols) { bad = true; continue; }
                    const uint32_t c = (uint32_t)col[j][i] - (uint32_t)base;
                    if (c >= bits_a_pass) continue;
                    if (c >> 5 != at) {
                        if (bits) atomicOr(&bm[at], bits);
                        at = c >> 5;
                        bits = 0u;
                    }
                    bits |= 1u << (c & 31u);
                }
                if (bits) atomicOr(&bm[at], bits);
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int j = threadIdx.x; j < words; j += NT) cnt += __popc(bm[j]);
        __syncthreads();
    }
    if (bad) atomicOr(p.ctl, 8);
    cnt = wave_sum(cnt);
    if ((threadIdx.x & 63) == 0) smem[threadIdx.x >> 6] = cnt;
    __syncthreads();
    int total = 0;
#pragma unroll 1
    for (int i = 0; i < NT / 64; ++i) total += smem[i];
    return total;
}

// windows of up to kCountTinyCap non-zeros, one workgroup each: all windows, or -- after a structural change -- the
// touched ones, whose larger members are listed for the kernels below
__global__ __launch_bounds__(256) void k_pre_count(Prep p)
{
    __shared__ int32_t table[2 * kCountTinyCap];
    __shared__ int smem[256 / 64];
    if (*p.ctl & 7) return;
    const int32_t w = p.touched ? p.touched[blockIdx.x] : (int32_t)blockIdx.x;
    const int32_t n = p.nnzw[w];
    if (n > kCountTinyCap) {
        if (p.touched && threadIdx.x == 0) {
            if (n > kCountMidCap) p.count_huge[atomicAdd(p.n_count_huge, 1)] = w;
            else if (n > kUniqueSmallCap) p.count_mid[atomicAdd(p.n_count_mid, 1)] = w;
            else p.count_1k[atomicAdd(p.ctl + 3, 1)] = w;
        }
        return;
    }
    int32_t s, e;
    window_span(w, p.n_rows, p.rowptr, s, e);
    const int nc = count_distinct(s, e, p, table, smem, threadIdx.x, 256);
    if (threadIdx.x == 0) p.ncols[w] = nc;
}

__global__ __launch_bounds__(256) void k_pre_count_1k(Prep p)
{
    __shared__ int32_t table[2 * kUniqueSmallCap];
    __shared__ int smem[256 / 64];
    if (*p.ctl & 7) return;
    const int32_t n = p.ctl[3];
    for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int32_t w = p.count_1k[i];
        int32_t s, e;
        window_span(w, p.n_rows, p.rowptr, s, e);
        const int nc = count_distinct(s, e, p, table, smem, threadIdx.x, 256);
        if (threadIdx.x == 0) p.ncols[w] = nc;
        __syncthreads();
    }
}

__global__ __launch_bounds__(1024) void k_pre_count_big(Prep p)
{
    __shared__ int32_t table[2 * kCountMidCap];
    __shared__ int smem[1024 / 64];
    if (*p.ctl & 7) return;
    const int32_t n_huge = *p.n_count_huge, n_mid = *p.n_count_mid, n_1k = p.big_takes_1k ? p.ctl[3] : 0;
    for (int32_t i = blockIdx.x; i < n_huge + n_mid + n_1k; i += gridDim.x) {
        const int32_t w = i < n_huge ? p.count_huge[i] : i < n_huge + n_mid ? p.count_mid[i - n_huge] : p.count_1k[i - n_huge - n_mid];
        int32_t s, e;
        window_span(w, p.n_rows, p.rowptr, s, e);
        const int nc = e - s <= kCountMidCap ? count_distinct(s, e, p, table, smem, threadIdx.x, 1024)
                                             : count_bits<1024>(s, e, p, reinterpret_cast<uint32_t*>(table), min((p.n_cols - 1) / 32 + 1, 2 * kCountMidCap), smem);
        if (threadIdx.x == 0) p.ncols[w] = nc;
        __syncthreads();
    }
}

// Few windows to count (all of a small matrix, or the touched ones): one launch for all sizes, where by class the larger
// windows wait for the small ones' launch and a few workgroups walk their list.  Windows of up to kCountTinyCap non-zeros take 256 threads each, two to a
// workgroup.  The larger ones, often neighbours, belong to the first n_big workgroups (few_big), every n_big-th window to each, which look for
// theirs among up to 32 and take them one by one with a bitmap.  LDS for that grows with the columns up to 32 KB (matrices of up to 2^20 columns: four passes).
// Bound by its longest chain of reads and by launches, so everything that does not depend on an answer from memory is asked for at once, and neither
// k_pre_validate (ALL) nor k_pre_select is launched.
// ALL: every window of the matrix, whose row offsets are checked here as well (k_pre_rows sums the windows itself); else the touched ones, whose sums go to
// their tiles from here.
// 16,934 rows: 9.3 us, and 3.0 and 3.8 for the two launches that are gone, -> 6.8 us; 1,000 touched windows of 169,343 rows: 27 -> 15 us, by the largest of
// them.  (Workgroups of 1024 threads and 64 KB, four windows each and the larger ones after the small: a CU's second workgroup starts 5 us late, and a hash set takes
// 6 us for 7,700 non-zeros.)  By class the same matrices took 3 to 10 us more, and 4,000 windows lose here: the line is at the windows that run at once.
constexpr int kFewWindows = 2048, kFewCols = 1 << 20, kFewThreads = 512, kFewBig = 64, kFewMostWords = 8192;
static_assert(kFewWindows <= 32 * kFewBig && kFewCols <= 4 * 32 * kFewMostWords, "windows to a workgroup, passes");
template <bool ALL>
__global__ __launch_bounds__(kFewThreads) void k_pre_count_few(Prep p, int32_t n_count, int32_t n_big, int words)
{
    constexpr int SMALL = kFewThreads / 256;
    extern __shared__ int32_t few_lds[];                        // SMALL * 2 * kCountTinyCap or `words`, whichever is more
    __shared__ int smem[kFewThreads / 64];
    const bool big = (int32_t)blockIdx.x < n_big;
    const int tid = threadIdx.x & 255, group = threadIdx.x >> 8;
    const int32_t i = big ? (int32_t)blockIdx.x + (int32_t)(threadIdx.x & 31) * n_big : ((int32_t)blockIdx.x - n_big) * SMALL + group;
    int32_t w = i >= n_count ? -1 : ALL ? i : p.touched[i], s, e;
    window_span(max(w, 0), p.n_rows, p.rowptr, s, e);
    if constexpr (ALL) {
        if (!big && w >= 0) {
            if (tid < kH) {
                const int64_t r = min((int64_t)w * kH + tid, (int64_t)p.n_rows - 1);
                const int32_t a = p.rowptr[r], b = p.rowptr[r + 1];
                if (a < 0 || b < a) atomicOr(p.ctl, 4);
            }
            if (tid == 0) {
                p.nnzw[w] = e - s;
                list_window(p, w, e - s, false);
            }
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            if (p.rowptr[0] != 0) atomicOr(p.ctl, 1);
            if ((int64_t)p.rowptr[p.n_rows] != p.nnz) atomicOr(p.ctl, 2);
        }
        // offsets that lead outside the arrays are an error by now, here or at the window that they belong to: nothing is read from there
        if (s < 0 || e < s || e > p.nnz) s = e = 0;
    } else if (*p.ctl & 7) {
        return;
    }
    if (w < 0) s = e = 0;
    auto counted = [&](int32_t window, int32_t n, int nc) {     // by one thread
        p.ncols[window] = nc;
        if constexpr (ALL) p.on_matrix[window] = window_route(p, p.mode, nc, n) ? n : 0;
        else
#pragma unroll 1
            for (int k = 0; k < 2; ++k) {                       // what the old count has added is taken off again
                unsigned long long v[kWt];
                const int32_t c = k == 0 ? p.old_ncols[window] : nc;
                window_sums(window_route(p, p.mode, c, n), c, n, v);
                add_to_tile(p, window, v, k == 0);
            }
    };
    if (!big) {
        const bool take = w >= 0 && e - s <= kCountTinyCap;
        if (!take) s = e = 0;
        const int nc = count_distinct(s, e, p, few_lds + group * 2 * kCountTinyCap, smem + group * 4, tid, 256);
        if (take && tid == 0) counted(w, e - s, nc);
        return;
    }
    // (every wave has all of the workgroup's windows in its lanes)
    uint32_t left = (uint32_t)__ballot(e - s > kCountTinyCap);
    while (left != 0) {
        const int q = __builtin_ctz(left);
        left &= left - 1;
        const int32_t cs = __builtin_amdgcn_readlane(s, q), ce = __builtin_amdgcn_readlane(e, q), cw = __builtin_amdgcn_readlane(w, q);
        __syncthreads();
        const int nc = count_bits<kFewThreads>(cs, ce, p, reinterpret_cast<uint32_t*>(few_lds), words, smem);
        if (threadIdx.x == 0) counted(cw, ce - cs, nc);
    }
}

__global__ __launch_bounds__(256) void k_pre_select(Prep p)
{
    const int tile = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (tile >= p.n_tiles) return;
    const int32_t w = tile * kTileWindows + (threadIdx.x & 63);
    unsigned long long v[kWt];
    const long long nc = w < p.W ? p.ncols[w] : 0, nz = w < p.W ? p.nnzw[w] : 0;
    window_sums(window_route(p, p.mode, nc, nz), nc, nz, v);
    if (*p.ctl) return;
#pragma unroll
    for (int i = 0; i < kWt; ++i) v[i] = wave_sum_u64(v[i]);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int i = 0; i < kWt; ++i) p.wt[(int64_t)tile * kWt + i] = v[i];
}

// Launch guard: a path whose share cannot repay a kernel launch of its own joins the other path.
__device__ inline int effective_mode(const Prep& p, unsigned long long on_matrix_)
{
    if (p.mode != HCSPMM_ROUTE_HYBRID) return p.mode;
    const int64_t on_matrix = (int64_t)on_matrix_, on_scalar = p.nnz - on_matrix;
    if (on_matrix > 0 && on_scalar > 0) {
        if (on_matrix < kGuardNnz && kGuardShare * on_matrix < p.nnz) return HCSPMM_ROUTE_ALL_CSR;
        if (on_scalar < kGuardNnz && kGuardShare * on_scalar < p.nnz) return HCSPMM_ROUTE_ALL_MFMA;
    }
    return p.mode;
}
__device__ inline int counts_set(const Prep& p, int mode)       // which set of the tile sums holds for the effective mode (-1: none)
{
    return mode == p.mode ? 0 : (mode == HCSPMM_ROUTE_ALL_MFMA ? 1 : -1);
}

// Whether every window runs on the scalar path (1) and in column panels (2), where panel_count or scalar_candidate ask.
//  * Panels fetch from L2 almost only, and pay where rows that run side by side do not find each other's X rows there anyway:
//    more than half of the columns of 65,536 consecutive non-zeros are distinct.  Against the plain scalar path, 64 columns,
//    fp32: power law, 200,000 rows of 300 (0.66): 1358 -> 1130 us, 100,000 of 200 (0.55): 357 -> 329 us, 120,000 of 150
//    (0.51): 302 -> 306 us, 60,000 of 150 (0.41 to 0.48): 130 -> 139 us; communities of 4,096 (0.10) and 32,768 (0.46) nodes:
//    776 -> 1090 us and 756 -> 980 us.  Rows of X off the 128-byte lines have no column slices to fall back on and take panels
//    from 0.4 on (60,000 of 150, 48 columns: 154 -> 134 us).  The matrix's rows must ascend.
//  * The plain scalar path takes over the matrix path's windows where the windows' distinct columns are more than 0.6 of their
//    non-zeros: the matrix path fetches a distinct column of a window once, the scalar path a row of X per non-zero but in
//    large part from L2.  They are 0.16 of them in communities of degree 51 (131,072 rows, 128 columns, fp32: 107 us on the
//    matrix path, 131 us on the scalar path) and 0.8 to 0.95 in power-law graphs of degree 20 to 500.  The whole matrix is
//    asked, not the matrix path's windows alone, because the two paths' stages follow each other: communities next to a
//    power law, 128 columns, per window / all scalar: 0.48 on the matrix path's windows, 0.63 on all: 792 / 723 us in fp32,
//    480 / 404 us in bf16; 0.16 and 0.75: 655 / 650 and 357 / 345 us; 0.16 and 0.61: 732 / 740 and 498 / 480 us.  At 256
//    columns they are level within 2 % (one of nine graphs, bf16: 1467 / 1563 us).
//    Where panels were asked for and neighbouring rows turn out to share, their X rows meet in L2 and the matrix may be of any
//    size (communities of 16,384, 60 M non-zeros, 128 columns, fp32: 2746 us on the matrix path, 2104 in panels, 1666 us).
__device__ inline int scalar_form(const Prep& p, int64_t total_ncols)
{
    const bool sample = p.panels_from > 0;
    const bool scattered = sample && 100 * (int64_t)p.ctl[8] > (int64_t)p.panels_from * kSamples * p.sample_len;
    if (scattered && p.ctl[6] == 0) return 2;
    return (p.scalar_exec || (sample && !scattered)) && p.features && 10 * total_ncols > 6 * p.nnz ? 1 : 0;
}

// One row's place in the scalar path's tables.
struct RowClass { int is_short, is_mid, n_seg, rest, len_long; };
__device__ inline RowClass row_class(const Prep& p, int32_t len, int route, int wide_window)
{
    RowClass c;
    const bool csr = route == 0, is_long = csr && len > p.long_row;
    c.is_mid = csr && !is_long && len > p.mid_row;
    c.is_short = csr && !is_long && !c.is_mid;
    c.n_seg = is_long ? (len + kSegLen - 1) / kSegLen : 0;
    // rows whose aggregated values reach memory even when the update stage is fused into the SpMM kernels: scalar-path
    // rows above the fused tier and all rows of matrix-path windows too wide for the wave-per-window kernel
    c.rest = csr ? len > p.fused_mid_row : wide_window;
    c.len_long = (is_long || c.is_mid) ? len : 0;
    return c;
}
// short | mid | rest | multi-segment rows, 16 bits each (a tile has 1024 rows); segments | partial rows, 32 bits each
__device__ inline unsigned long long row_counts(const RowClass& c)
{
    return (unsigned long long)c.is_short | (unsigned long long)c.is_mid << 16 | (unsigned long long)c.rest << 32 |
           (unsigned long long)(c.n_seg > 1) << 48;
}
__device__ inline unsigned long long seg_counts(const RowClass& c)
{
    return (unsigned long long)c.n_seg | (unsigned long long)(c.n_seg > 1 ? c.n_seg : 0) << 32;
}

// Both kernels of the rows are a few trips to memory and sums over the workgroup: what does not depend on an answer is asked for first, and sums are DPP moves
// (169,343 rows: 6.3 and 7.5 us with shuffles and one trip after the other, 4.9 and 5.7 so; with a thread per row, 16 waves to a CU that wait for each other at every
// sum, 6.7 and 11).
// DIRECT: up to kFewWindows windows, whose sums every workgroup forms itself, and those of its own tile for the kernels behind it.
template <bool DIRECT>
__global__ __launch_bounds__(256) void k_pre_rows(Prep p)
{
    __shared__ unsigned long long smem[4 * 4];
    __shared__ uint8_t s_route[kTileWindows], s_wide[kTileWindows];
    const int tile = blockIdx.x, t = threadIdx.x;
    const int64_t i0 = min((int64_t)tile * kTileRows + 4 * t, (int64_t)p.n_rows);
    int32_t start[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) start[j] = p.rowptr[min(i0 + j, (int64_t)p.n_rows)];
    const int32_t w = tile * kTileWindows + (t & 63);
    const long long nc = w < p.W ? p.ncols[w] : 0, nz = w < p.W ? p.nnzw[w] : 0;
    const int own = window_route(p, p.mode, nc, nz);            // under the plan's own mode
    unsigned long long all[3] = {0, 0, 0};                      // columns in front of the tile, from it on; non-zeros on the matrix path
    if constexpr (DIRECT) {
        int32_t c[kFewWindows / 256], on[kFewWindows / 256];
#pragma unroll
        for (int j = 0; j < kFewWindows / 256; ++j) {
            const int32_t i = min(t + 256 * j, p.W - 1);
            c[j] = p.ncols[i];
            on[j] = p.on_matrix[i];
        }
        if (*p.ctl) return;
#pragma unroll
        for (int j = 0; j < kFewWindows / 256; ++j) {
            const int32_t i = t + 256 * j;
            if (i >= p.W) break;
            all[2] += (unsigned long long)on[j];
            all[i < tile * kTileWindows ? 0 : 1] += (unsigned long long)c[j];
        }
        unsigned long long v[kWt];                              // two of the tile's sums to a wave
        window_sums(own, nc, nz, v);
        const int wave = t >> 6;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const unsigned long long sum = wave_sum_u64(wave == 0 ? v[i] : wave == 1 ? v[2 + i] : wave == 2 ? v[4 + i] : v[6 + i]);
            if ((t & 63) == 0) p.wt[(int64_t)tile * kWt + 2 * wave + i] = sum;
        }
    } else {
        for_sums<kWt, true>(p.wt, p.wg, p.n_tiles, tile, t, 256, [&](const unsigned long long* v, bool in_front) {
            all[2] += v[1];
            all[in_front ? 0 : 1] += v[0];
        });
        if (*p.ctl) return;
    }
    block_sums_u64<3>(all, smem);
    const int mode = effective_mode(p, all[2]);
    if (t < kTileWindows) {
        const int r = mode == p.mode ? own : mode == HCSPMM_ROUTE_ALL_MFMA && nc > 0;
        s_route[t] = (uint8_t)r;
        s_wide[t] = nc > kMfmaSmallMaxCols ? 1 : 0;
        const unsigned long long inc = wave_scan_u64((unsigned long long)nc);
        if (w < p.W) {
            p.route[w] = (uint8_t)r;
            p.wptr[w] = (int64_t)(all[0] + inc - (unsigned long long)nc);
            if (w == p.W - 1) p.wptr[p.W] = (int64_t)(all[0] + inc);
        }
        if (p.W == 0 && t == 0) p.wptr[0] = 0;
    }
    __syncthreads();
    const int all_scalar = scalar_form(p, (int64_t)(all[0] + all[1]));
    if (tile == 0 && t == 0) p.ctl[7] = all_scalar;
    const int route = all_scalar != 0 ? 0 : s_route[t / (kH / 4)], wide = s_wide[t / (kH / 4)];
    unsigned long long sum[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (i0 + j >= p.n_rows) break;
        const RowClass c = row_class(p, start[j + 1] - start[j], route, wide);
        sum[0] += (unsigned long long)c.is_short | (unsigned long long)c.is_mid << 32;
        sum[1] += (unsigned long long)c.rest | (unsigned long long)(c.n_seg > 1) << 32;
        sum[2] += seg_counts(c);
        sum[3] += (unsigned long long)c.len_long;
    }
    block_sums_u64<4>(sum, smem);
    if (t == 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) p.rt[(int64_t)tile * kRt + i] = sum[i];
}

// Fills the row tables whose pointers are set; one workgroup behind the last tile's writes the totals (when p.out is set).
__global__ __launch_bounds__(256) void k_pre_fill(Prep p)
{
    __shared__ unsigned long long smem[4 * 11];
    const int tile = blockIdx.x, t = threadIdx.x;
    const bool last = tile == p.n_tiles;
    const int64_t i0 = min((int64_t)tile * kTileRows + 4 * t, (int64_t)p.n_rows);
    const int32_t w = (int32_t)(i0 / kH);
    int32_t start[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) start[j] = p.rowptr[min(i0 + j, (int64_t)p.n_rows)];
    const int32_t own_route = w < p.W ? p.route[w] : 0, own_cols = w < p.W ? p.ncols[w] : 0;
    unsigned long long front[3] = {0, 0, 0};                    // short | mid, rest | multi, segments | partial rows in front of the tile
    for_sums<kRt, false>(p.rt, p.rg, p.n_tiles, tile, t, 256, [&](const unsigned long long* v, bool) { front[0] += v[0]; front[1] += v[1]; front[2] += v[2]; });
    unsigned long long v[11] = {};                              // the last workgroup's: distinct columns, long rows' non-zeros; the tiles' sums of windows in both sets
    if (last && p.out) {
        for_sums<kRt, true>(p.rt, p.rg, p.n_tiles, p.n_tiles, t, 256, [&](const unsigned long long* u, bool) { v[1] += u[3]; });
        for_sums<kWt, true>(p.wt, p.wg, p.n_tiles, p.n_tiles, t, 256, [&](const unsigned long long* u, bool) {
            v[0] += u[0];
            v[6] += u[7];
#pragma unroll
            for (int set = 0; set < 2; ++set) {
                const unsigned long long n = u[2 + 3 * set];
                v[2 + 5 * set] += u[1 + 3 * set];
                v[3 + 5 * set] += (n & 0xffffull) | (n >> 16 & 0xffffull) << 32;
                v[4 + 5 * set] += (n >> 32 & 0xffffull) | (n >> 48) << 32;
                v[5 + 5 * set] += u[3 + 3 * set];
            }
        });
    }
    const int32_t all_scalar = p.ctl[7];
    if (*p.ctl) {
        if (last && t == 0 && p.out) p.out->err = *p.ctl;
        return;
    }
    block_sums_u64<3>(front, smem);
    const unsigned long long sm = front[0], rm = front[1], seg = front[2];
    const int route = all_scalar == 0 ? own_route : 0, wide = own_cols > kMfmaSmallMaxCols ? 1 : 0;
    RowClass c[4];
    unsigned long long at[2] = {0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        c[j] = RowClass{0, 0, 0, 0, 0};
        if (i0 + j < p.n_rows) c[j] = row_class(p, start[j + 1] - start[j], route, wide);
        at[0] += row_counts(c[j]);
        at[1] += seg_counts(c[j]);
    }
    block_scans_u64<2>(at, smem);
    uint32_t n_short = (uint32_t)sm + (uint32_t)(at[0] & 0xffffull), n_mid = (uint32_t)(sm >> 32) + (uint32_t)(at[0] >> 16 & 0xffffull);
    uint32_t n_rest = (uint32_t)rm + (uint32_t)(at[0] >> 32 & 0xffffull), n_multi = (uint32_t)(rm >> 32) + (uint32_t)(at[0] >> 48);
    uint32_t n_seg = (uint32_t)seg + (uint32_t)at[1], n_slot = (uint32_t)(seg >> 32) + (uint32_t)(at[1] >> 32);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int32_t i = (int32_t)(i0 + j);
        if (c[j].is_short) { if (p.short_rows) p.short_rows[n_short] = i; ++n_short; }
        if (c[j].is_mid) { if (p.mid_rows) p.mid_rows[n_mid] = i; ++n_mid; }
        if (c[j].rest) { if (p.rest_rows) p.rest_rows[n_rest] = i; ++n_rest; }
        const int ns = c[j].n_seg;
        if (ns == 0) continue;
        if (p.segs)
#pragma unroll 1
            for (int q = 0; q < ns; ++q) {
                Segment sg;
                sg.row = i;
                sg.k_begin = start[j] + q * kSegLen;
                sg.k_end = min(start[j + 1], sg.k_begin + kSegLen);
                sg.slot = ns > 1 ? (int32_t)(n_slot + q) : -1;
                p.segs[n_seg + q] = sg;
            }
        n_seg += ns;
        if (ns > 1) {
            if (p.multi) {
                MultiRow m;
                m.row = i; m.first_slot = (int32_t)n_slot; m.n_slots = ns; m.pad = 0;
                p.multi[n_multi] = m;
            }
            ++n_multi;
            n_slot += ns;
        }
    }
    if (!last || !p.out) return;
    // what is in front of the place behind the last tile are the row totals
    block_sums_u64<11>(v, smem);
    const int set = counts_set(p, effective_mode(p, v[2]));
    if (t == 0) {
        PrepTotals o{};
        o.total_ncols = (int64_t)v[0]; o.nnz_long = (int64_t)v[1];
        if (set >= 0) {
            const unsigned long long lo = set == 0 ? v[3] : v[8], hi = set == 0 ? v[4] : v[9];
            o.nnz_mfma = (int64_t)(set == 0 ? v[2] : v[7]); o.wide_cols = (int64_t)(set == 0 ? v[5] : v[10]); o.mfma_cols = (int64_t)(set == 0 ? v[6] : v[0]);
            o.n_mfma = (int32_t)lo; o.n_mfma_small = (int32_t)(lo >> 32);
            o.n_mfma_mid = (int32_t)hi; o.n_mfma_big = (int32_t)(hi >> 32);
        }
        o.n_short = (int32_t)n_short; o.n_mid = (int32_t)n_mid; o.n_rest = (int32_t)n_rest; o.n_multi = (int32_t)n_multi;
        o.n_segs = (int32_t)n_seg; o.n_slots = (int64_t)n_slot;
        o.n_big_list = p.ctl[1]; o.n_huge_list = p.ctl[2];
        o.all_scalar = p.ctl[7];
        o.sample_distinct = p.ctl[8];
        o.err = 0;
        *p.out = o;
    }
}

// ascending lists of the matrix path's windows, all and per kernel
__global__ __launch_bounds__(256) void k_pre_windows(Prep p, int32_t* __restrict__ mfma, int32_t* __restrict__ small,
                                                     int32_t* __restrict__ mid, int32_t* __restrict__ big)
{
    const int tile = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (tile >= p.n_tiles) return;
    unsigned long long on_matrix = 0, lo = 0, hi = 0;           // matrix | small, medium | wide windows in front of the tile
    for_sums<kWt, true>(p.wt, p.wg, p.n_tiles, tile, lane, 64, [&](const unsigned long long* v, bool) { on_matrix += v[1]; });
    const int set = counts_set(p, effective_mode(p, wave_sum(on_matrix)));
    if (set >= 0)
        for_sums<kWt, false>(p.wt, p.wg, p.n_tiles, tile, lane, 64, [&](const unsigned long long* v, bool) {
            const unsigned long long n = v[2 + 3 * set];
            lo += (n & 0xffffull) | (n >> 16 & 0xffffull) << 32;
            hi += (n >> 32 & 0xffffull) | (n >> 48) << 32;
        });
    lo = wave_sum(lo);
    hi = wave_sum(hi);
    const int32_t w = tile * kTileWindows + lane;
    const int r = w < p.W ? p.route[w] : 0;
    const unsigned long long n = w < p.W ? window_counts(r, p.ncols[w]) : 0;
    unsigned long long inc = n;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long t = __shfl_up(inc, off, 64);
        if (lane >= off) inc += t;
    }
    if (w >= p.W) return;
    const unsigned long long ex = inc - n;
    const uint32_t i_mfma = (uint32_t)lo + (uint32_t)(ex & 0xffffull);
    if (!r) return;
    mfma[i_mfma] = w;
    if (n >> 16 & 0xffffull) small[(uint32_t)(lo >> 32) + (uint32_t)(ex >> 16 & 0xffffull)] = w;
    else if (n >> 32 & 0xffffull) mid[(uint32_t)hi + (uint32_t)(ex >> 32 & 0xffffull)] = w;
    else big[(uint32_t)(hi >> 32) + (uint32_t)(ex >> 48)] = w;
}

// How many of k_pre_count_few's workgroups are for the larger windows, by the matrix's non-zeros per window.  Each counts its own one by one, so graphs whose windows are
// mostly large want many (64 / 256 / 512 of them, whole calls, us, power laws: 9,913 rows of 210: 100.9 / 85.3 / 82.7, 20,000 of 120: 84.0 / 68.5 / 66.1, 100,000
// of 100 with 700 rows changed: 248 / 226 / 226; 32,000 of 60: 74.4 / 64.1 / 64.3, 8,000 of 60: 52.8 / 52.0 / 52.8), others few, since every one looks for its own before
// it may leave (16,934 of 14: 57.2 / 57.5 / 57.7).
static int32_t few_big(const Prep& p)
{
    return p.nnz <= 256 * (int64_t)p.W ? kFewBig : p.nnz <= 1024 * (int64_t)p.W ? 4 * kFewBig : 8 * kFewBig;
}

// Whether k_pre_count_few counts the windows.
static bool prep_counts_few(const Prep& p, int32_t n_touched)
{
    const int64_t n_count = p.touched ? n_touched : p.W;
    return p.features && n_count > 0 && n_count <= kFewWindows && p.n_cols <= kFewCols;
}
size_t prep_zeros(const Prep& p, int32_t n_touched) { return p.touched && prep_counts_few(p, n_touched) ? (size_t)kWt * p.n_tiles * sizeof(unsigned long long) : 0; }

hipError_t launch_prep(const Prep& p_, int32_t n_touched, hipStream_t s)
{
    Prep p = p_;
    const int64_t n_count = p.touched ? n_touched : p.W;
    const bool few = prep_counts_few(p, n_touched);
    p.big_takes_1k = n_count <= kBigTakes1kWindows ? 1 : 0;
    if (few) p.on_matrix = p.count_1k;                          // k_pre_count_few has no lists
    const dim3 grid_rows((unsigned)(((int64_t)p.n_rows + 1 + 255) / 256));
    if (few && p.touched) hipLaunchKernelGGL(k_pre_validate<true>, grid_rows, dim3(256), 0, s, p);
    else if (!few) hipLaunchKernelGGL(k_pre_validate<false>, grid_rows, dim3(256), 0, s, p);
    if (p.features && p.W > 0) {
        if (few) {
            constexpr int per = kFewThreads / 256;
            const int words = std::min((p.n_cols - 1) / 32 + 1, kFewMostWords);
            const size_t lds = (size_t)std::max(words, per * 2 * kCountTinyCap) * sizeof(int32_t);
            const int32_t n_big = (int32_t)std::min<int64_t>(n_count, few_big(p));
            const dim3 grid((unsigned)(n_big + (n_count + per - 1) / per));
            if (p.touched) hipLaunchKernelGGL(k_pre_count_few<false>, grid, dim3(kFewThreads), lds, s, p, (int32_t)n_count, n_big, words);
            else hipLaunchKernelGGL(k_pre_count_few<true>, grid, dim3(kFewThreads), lds, s, p, (int32_t)n_count, n_big, words);
        } else {
            if (n_count > 0) hipLaunchKernelGGL(k_pre_count, dim3((unsigned)n_count), dim3(256), 0, s, p);
            // windows beyond the small set's capacity; how many there are only the device knows, so the grids are bounded by
            // what the matrix can hold and walk the lists
            auto most = [&](int64_t cap, int64_t limit) { return (unsigned)std::min<int64_t>({n_count, p.nnz / (cap + 1), limit}); };
            // (up to kBigTakes1kWindows windows to count: one launch serves both larger classes)
            const int64_t cap_big = p.big_takes_1k ? kCountTinyCap : kUniqueSmallCap;
            if (!p.big_takes_1k && most(kCountTinyCap, 2048) > 0)
                hipLaunchKernelGGL(k_pre_count_1k, dim3(most(kCountTinyCap, 2048)), dim3(256), 0, s, p);
            if (most(cap_big, 256) > 0) hipLaunchKernelGGL(k_pre_count_big, dim3(most(cap_big, 256)), dim3(1024), 0, s, p);
        }
    } else if (p.nnz > 0) {
        int64_t blocks = (p.nnz + 256 * 8 - 1) / (256 * 8);
        if (blocks > 65536) blocks = 65536;
        const int samples = p.sample_len > 0 && p.panels_from == 0 ? kSamples : 0;
        hipLaunchKernelGGL(k_validate_cols, dim3((unsigned)(blocks + samples)), dim3(256), 0, s, p, samples);
    }
    if (p.panels_from > 0) {
        hipLaunchKernelGGL(k_pre_sample, dim3(kSamples), dim3(1024), 0, s, p);
        int64_t blocks = (p.nnz + 256 * 16 - 1) / (256 * 16);
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(k_pre_sorted, dim3((unsigned)blocks), dim3(256), 0, s, p);
    }
    if (!few) hipLaunchKernelGGL(k_pre_select, dim3((unsigned)(p.n_tiles + 3) / 4), dim3(256), 0, s, p);
    const int32_t groups = group_count(p.n_tiles);
    if (groups) hipLaunchKernelGGL(k_group_sums<kWt>, dim3((unsigned)groups), dim3(256), 0, s, p.n_tiles, p.wt, p.wg);
    if (few && !p.touched) hipLaunchKernelGGL(k_pre_rows<true>, dim3((unsigned)p.n_tiles), dim3(256), 0, s, p);
    else hipLaunchKernelGGL(k_pre_rows<false>, dim3((unsigned)p.n_tiles), dim3(256), 0, s, p);
    if (groups) hipLaunchKernelGGL(k_group_sums<kRt>, dim3((unsigned)groups), dim3(256), 0, s, p.n_tiles, p.rt, p.rg);
    hipLaunchKernelGGL(k_pre_fill, dim3((unsigned)p.n_tiles + 1), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_prep_fill(const Prep& p, hipStream_t s)
{
    hipLaunchKernelGGL(k_pre_fill, dim3((unsigned)p.n_tiles), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_prep_windows(const Prep& p, int32_t* mfma, int32_t* small, int32_t* mid, int32_t* big, hipStream_t s)
{
    hipLaunchKernelGGL(k_pre_windows, dim3((unsigned)(p.n_tiles + 3) / 4), dim3(256), 0, s, p, mfma, small, mid, big);
    return hipGetLastError();
}

// Which matrix-path windows keep the previous plan's condensed structure: on that path before and now, and not
// touched.  todo[w] is the route restricted to the windows that still have to be condensed.
__global__ __launch_bounds__(256) void k_carry_mask(int32_t W, const uint8_t* __restrict__ old_route,
                                                    const uint8_t* __restrict__ route, uint8_t* __restrict__ carried,
                                                    uint8_t* __restrict__ todo)
{
    const int32_t w = blockIdx.x * 256 + threadIdx.x;
    if (w >= W) return;
    const uint8_t c = (old_route[w] != 0 && route[w] != 0) ? 1 : 0;
    carried[w] = c;
    todo[w] = (route[w] != 0 && !c) ? 1 : 0;
}

__global__ __launch_bounds__(256) void k_carry_untouch(int32_t n_touched, const int32_t* __restrict__ touched,
                                                       const uint8_t* __restrict__ route, uint8_t* __restrict__ carried,
                                                       uint8_t* __restrict__ todo)
{
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n_touched) return;
    const int32_t w = touched[i];
    carried[w] = 0;
    todo[w] = route[w] != 0 ? 1 : 0;
}

// Copies a carried window's column list and the condensed columns of its non-zeros from the previous plan's arrays
// to their new places (both move when windows in front of it changed size).
__global__ __launch_bounds__(256) void k_carry_copy(int32_t n_rows, const uint8_t* __restrict__ carried,
                                                    const int64_t* __restrict__ old_wptr, const int64_t* __restrict__ wptr,
                                                    const int32_t* __restrict__ old_wcols, int32_t* __restrict__ wcols,
                                                    const int64_t* __restrict__ old_start, const int32_t* __restrict__ rowptr,
                                                    const int32_t* __restrict__ old_erc, int32_t* __restrict__ erc)
{
    const int32_t w = blockIdx.x;
    if (!carried[w]) return;
    const int64_t so = old_wptr[w], sn = wptr[w];
    const int32_t nc = (int32_t)(wptr[w + 1] - sn);
    for (int32_t i = threadIdx.x; i < nc; i += 256) wcols[sn + i] = old_wcols[so + i];
    int32_t s, e;
    window_span(w, n_rows, rowptr, s, e);
    const int64_t eo = old_start[w];
    for (int32_t k = threadIdx.x; k < e - s; k += 256) erc[s + k] = old_erc[eo + k];
}

hipError_t launch_carry_mask(int32_t W, const uint8_t* old_route, const uint8_t* route, int32_t n_touched,
                             const int32_t* touched, uint8_t* carried, uint8_t* todo, hipStream_t s)
{
    if (W <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_carry_mask, dim3((W + 255) / 256), dim3(256), 0, s, W, old_route, route, carried, todo);
    if (n_touched > 0)
        hipLaunchKernelGGL(k_carry_untouch, dim3((n_touched + 255) / 256), dim3(256), 0, s, n_touched, touched, route,
                           carried, todo);
    return hipGetLastError();
}

hipError_t launch_carry_copy(int32_t W, int32_t n_rows, const uint8_t* carried, const int64_t* old_wptr, const int64_t* wptr,
                             const int32_t* old_wcols, int32_t* wcols, const int64_t* old_start, const int32_t* rowptr,
                             const int32_t* old_erc, int32_t* erc, hipStream_t s)
{
    if (W <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_carry_copy, dim3(W), dim3(256), 0, s, n_rows, carried, old_wptr, wptr, old_wcols, wcols, old_start,
                       rowptr, old_erc, erc);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// compact the distinct-column lists and give every non-zero its condensed column
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_ecol(int32_t n_rows, const int32_t* __restrict__ rowptr,
                                              const int32_t* __restrict__ colind,
                                              const int32_t* __restrict__ tmp_cols, const int32_t* __restrict__ ncols,
                                              const int64_t* __restrict__ wptr, int32_t* __restrict__ wcols,
                                              int32_t* __restrict__ erc, int32_t* __restrict__ unsorted_flag,
                                              const uint8_t* __restrict__ route, int want, int32_t skip_above)
{
    __shared__ int32_t ucols[kEcolLdsCap];
    __shared__ int32_t rp[kH + 1];
    const int32_t w = blockIdx.x;
    if ((route[w] != 0) != (want != 0)) return;      // only the windows of one route
    int32_t s, e;
    window_span(w, n_rows, rowptr, s, e);
    if (e == s || e - s > skip_above) return;        // larger windows were condensed by k_condense_rank
    const int32_t nc = ncols[w];
    const int64_t wp = wptr[w];
    const int32_t* __restrict__ src = tmp_cols + (int64_t)s;
    if (threadIdx.x <= kH) {
        int64_t r = (int64_t)w * kH + threadIdx.x;
        if (r > n_rows) r = n_rows;
        rp[threadIdx.x] = rowptr[r];
    }
    const bool in_lds = nc <= kEcolLdsCap;
    for (int i = threadIdx.x; i < nc; i += 256) {
        int32_t c = src[i];
        wcols[wp + i] = c;
        if (in_lds) ucols[i] = c;
    }
    __syncthreads();
    for (int32_t k = s + threadIdx.x; k < e; k += 256) {
        const int32_t c = colind[k];
        int lo = 0, hi = nc - 1;               // c is in the list by construction
        if (in_lds) {
            while (lo < hi) { int mid = (lo + hi) >> 1; if (ucols[mid] < c) lo = mid + 1; else hi = mid; }
        } else {
            while (lo < hi) { int mid = (lo + hi) >> 1; if (src[mid] < c) lo = mid + 1; else hi = mid; }
        }
        int r = 0;                              // row of k inside the window: last r with rp[r] <= k
#pragma unroll
        for (int step = 8; step > 0; step >>= 1)
            if (r + step < kH && rp[r + step] <= k) r += step;
        erc[k] = (lo << 4) | r;
        // note rows whose column indices are not non-decreasing (the matrix path's cursor walk needs them sorted)
        if (k > rp[r] && colind[k - 1] > c) atomicOr(unsorted_flag, 1);
    }
}

hipError_t launch_ecol(int32_t W, int32_t n_rows, const int32_t* rowptr, const int32_t* colind,
                       const int32_t* tmp_cols, const int32_t* ncols, const int64_t* wptr, int32_t* wcols,
                       int32_t* erc, int32_t* unsorted_flag, const uint8_t* route, int want, int32_t skip_above,
                       hipStream_t s)
{
    hipLaunchKernelGGL(k_ecol, dim3(W), dim3(256), 0, s, n_rows, rowptr, colind, tmp_cols, ncols, wptr, wcols, erc,
                       unsorted_flag, route, want, skip_above);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// condensing of large matrix-path windows in one go: an LDS bitmap of the window's columns plus a
// prefix count per bitmap word gives the sorted list AND every non-zero's position in it (its rank)
// without a search; 2^19 columns per pass over the window's own column range
// ------------------------------------------------------------------------------------------------
constexpr int kRankWords = 16384;

__global__ __launch_bounds__(1024) void k_condense_rank(const int32_t* __restrict__ list, int32_t n_rows,
                                                        const int32_t* __restrict__ rowptr,
                                                        const int32_t* __restrict__ colind,
                                                        const uint8_t* __restrict__ route,
                                                        const int64_t* __restrict__ wptr, int32_t* __restrict__ wcols,
                                                        int32_t* __restrict__ erc, int32_t* __restrict__ unsorted_flag)
{
    __shared__ uint32_t bm[kRankWords];
    __shared__ int32_t pre[kRankWords];
    __shared__ int smem[1024 / 64 + 1];
    __shared__ int32_t rp[kH + 1];
    __shared__ int32_t span_lo, span_hi;
    constexpr int kBits = kRankWords * 32;
    const int32_t w = list[blockIdx.x];
    if (route[w] == 0) return;
    int32_t s, e;
    window_span(w, n_rows, rowptr, s, e);
    if (e == s) return;
    const int64_t wp = wptr[w];
    if (threadIdx.x <= kH) {
        int64_t r = (int64_t)w * kH + threadIdx.x;
        if (r > n_rows) r = n_rows;
        rp[threadIdx.x] = rowptr[r];
    }
    if (threadIdx.x == 0) { span_lo = 0x7fffffff; span_hi = -1; }
    __syncthreads();
    {
        int32_t lo = 0x7fffffff, hi = -1;
        for (int32_t k = s + threadIdx.x; k < e; k += 1024) {
            const int32_t c = colind[k];
            lo = min(lo, c);
            hi = max(hi, c);
        }
        if (hi >= 0) { atomicMin(&span_lo, lo); atomicMax(&span_hi, hi); }
    }
    __syncthreads();
    const int32_t cmax = span_hi;
    int32_t running = 0;
    for (int64_t base = span_lo & ~31; base <= cmax; base += kBits) {
        // words of this pass that can hold a column of the window, dealt to the threads in equal consecutive runs
        const int n_words = (int)min((int64_t)kRankWords, (cmax - base) / 32 + 1);
        const int wpt = (n_words + 1023) / 1024;
        const int w0 = threadIdx.x * wpt;
        for (int i = threadIdx.x; i < n_words; i += 1024) bm[i] = 0u;
        __syncthreads();
        for (int32_t k = s + threadIdx.x; k < e; k += 1024) {
            const int64_t c = (int64_t)colind[k] - base;
            if (c >= 0 && c < kBits) atomicOr(&bm[c >> 5], 1u << (c & 31));
        }
        __syncthreads();
        const int my_words = max(0, min(wpt, n_words - w0));
        int cnt = 0;
        for (int i = 0; i < my_words; ++i) cnt += __popc(bm[w0 + i]);
        int total;
        const int off = block_exclusive_scan<1024>(cnt, &total, smem);
        {
            int run = off;
            int32_t* out = wcols + wp + running + off;
            for (int i = 0; i < my_words; ++i) {
                uint32_t bits = bm[w0 + i];
                pre[w0 + i] = run;
                run += __popc(bits);
                while (bits) {
                    const int b = __ffs(bits) - 1;
                    bits &= bits - 1;
                    *out++ = (int32_t)(base + (int64_t)(w0 + i) * 32 + b);
                }
            }
        }
        __syncthreads();
        for (int32_t k = s + threadIdx.x; k < e; k += 1024) {
            const int32_t col = colind[k];
            const int64_t c = (int64_t)col - base;
            if (c < 0 || c >= kBits) continue;
            const int word = (int)(c >> 5);
            const int rank = running + pre[word] + __popc(bm[word] & ((1u << (c & 31)) - 1u));
            int r = 0;                              // row of k inside the window: last r with rp[r] <= k
#pragma unroll
            for (int step = 8; step > 0; step >>= 1)
                if (r + step < kH && rp[r + step] <= k) r += step;
            erc[k] = (rank << 4) | r;
            if (k > rp[r] && colind[k - 1] > col) atomicOr(unsorted_flag, 1);
        }
        running += total;
        __syncthreads();
    }
}

hipError_t launch_condense_rank(int32_t n_list, const int32_t* list, int32_t n_rows, const int32_t* rowptr,
                                const int32_t* colind, const uint8_t* route, const int64_t* wptr, int32_t* wcols,
                                int32_t* erc, int32_t* unsorted_flag, hipStream_t s)
{
    if (n_list <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_condense_rank, dim3(n_list), dim3(1024), 0, s, list, n_rows, rowptr, colind, route, wptr, wcols,
                       erc, unsorted_flag);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// runs of matrix-path windows: the union of the windows' column lists and every window column's
// position in it, by the same bitmap ranks (the lists are ascending, the union comes out ascending)
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_run_union(const int32_t* __restrict__ win_list, int32_t n_list,
                                                    const int32_t* __restrict__ ncols, const int64_t* __restrict__ wptr,
                                                    const int32_t* __restrict__ wcols, int32_t* __restrict__ ucols,
                                                    int32_t* __restrict__ wslot, RunDesc* __restrict__ runs)
{
    __shared__ uint32_t bm[kRankWords];
    __shared__ int32_t pre[kRankWords];
    __shared__ int smem[1024 / 64 + 1];
    constexpr int kBits = kRankWords * 32;
    constexpr int kWordsPerThread = kRankWords / 1024;
    const int32_t first = blockIdx.x * kRunWindows;
    const int nw = min(kRunWindows, n_list - first);
    int64_t wp[kRunWindows];
    int32_t nc[kRunWindows];
    int32_t lo = 0x7fffffff, hi = -1;
    for (int i = 0; i < nw; ++i) {
        const int32_t w = win_list[first + i];
        wp[i] = wptr[w];
        nc[i] = ncols[w];
        if (nc[i] > 0) {
            lo = min(lo, wcols[wp[i]]);
            hi = max(hi, wcols[wp[i] + nc[i] - 1]);
        }
    }
    const int64_t up = wp[0];                                  // the union is stored where the run's first window's list starts
    int32_t running = 0;
    const int w0 = threadIdx.x * kWordsPerThread;
    for (int64_t base = lo & ~31; base <= hi; base += kBits) {
        for (int i = threadIdx.x; i < kRankWords; i += 1024) bm[i] = 0u;
        __syncthreads();
        for (int i = 0; i < nw; ++i)
            for (int32_t k = threadIdx.x; k < nc[i]; k += 1024) {
                const int64_t c = (int64_t)wcols[wp[i] + k] - base;
                if (c >= 0 && c < kBits) atomicOr(&bm[c >> 5], 1u << (c & 31));
            }
        __syncthreads();
        int cnt = 0;
#pragma unroll 4
        for (int i = 0; i < kWordsPerThread; ++i) cnt += __popc(bm[w0 + i]);
        int total;
        const int off = block_exclusive_scan<1024>(cnt, &total, smem);
        {
            int run = off;
            int32_t* out = ucols + up + running + off;
            for (int i = 0; i < kWordsPerThread; ++i) {
                uint32_t bits = bm[w0 + i];
                pre[w0 + i] = run;
                run += __popc(bits);
                while (bits) {
                    const int b = __ffs(bits) - 1;
                    bits &= bits - 1;
                    *out++ = (int32_t)(base + (int64_t)(w0 + i) * 32 + b);
                }
            }
        }
        __syncthreads();
        for (int i = 0; i < nw; ++i)
            for (int32_t k = threadIdx.x; k < nc[i]; k += 1024) {
                const int64_t c = (int64_t)wcols[wp[i] + k] - base;
                if (c < 0 || c >= kBits) continue;
                const int word = (int)(c >> 5);
                wslot[wp[i] + k] = running + pre[word] + __popc(bm[word] & ((1u << (c & 31)) - 1u));
            }
        running += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        RunDesc rd;
        rd.up = up; rd.first = first; rd.nw = nw; rd.nu = running;
        rd.n_slices = 1; rd.slot0 = 0; rd.pad = 0;              // slices are laid out by the host from the union sizes
        runs[blockIdx.x] = rd;
    }
}

// per slice and wave: the window the wave owns, with what the kernel needs to start on it
__global__ __launch_bounds__(256) void k_run_wins(int32_t n_slices, const RunSlice* __restrict__ slices,
                                                  const RunDesc* __restrict__ runs, const int32_t* __restrict__ win_list,
                                                  const int32_t* __restrict__ ncols, const int64_t* __restrict__ wptr,
                                                  int32_t n_rows, const int32_t* __restrict__ rowptr, RunWin* __restrict__ wins)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n_slices * kRunWindows) return;
    const RunDesc rd = runs[slices[t / kRunWindows].run];
    const int i = (int)(t % kRunWindows);
    const int32_t w = win_list[rd.first + (i < rd.nw ? i : 0)];
    RunWin rw;
    rw.w = w; rw.nc = ncols[w]; rw.wp = wptr[w]; rw.pad = 0;
    rw.k_last = rowptr[min((int64_t)w * kH + kH, (int64_t)n_rows)] - 1;
    wins[t] = rw;
}

hipError_t launch_run_wins(int32_t n_slices, const RunSlice* slices, const RunDesc* runs, const int32_t* win_list,
                           const int32_t* ncols, const int64_t* wptr, int32_t n_rows, const int32_t* rowptr, RunWin* wins,
                           hipStream_t s)
{
    if (n_slices <= 0) return hipSuccess;
    const int64_t n = (int64_t)n_slices * kRunWindows;
    hipLaunchKernelGGL(k_run_wins, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n_slices, slices, runs, win_list, ncols,
                       wptr, n_rows, rowptr, wins);
    return hipGetLastError();
}

hipError_t launch_run_union(int32_t n_runs, const int32_t* win_list, int32_t n_list, const int32_t* ncols,
                            const int64_t* wptr, const int32_t* wcols, int32_t* ucols, int32_t* wslot, RunDesc* runs,
                            hipStream_t s)
{
    if (n_runs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_run_union, dim3(n_runs), dim3(1024), 0, s, win_list, n_list, ncols, wptr, wcols, ucols, wslot,
                       runs);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// matrix-path launch table: one descriptor per wave-per-window item
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_build_desc(int32_t n_list, const int32_t* __restrict__ win_list,
                                                    int32_t n_rows, const int32_t* __restrict__ rowptr,
                                                    const int32_t* __restrict__ ncols,
                                                    const int64_t* __restrict__ wptr, WinDesc* __restrict__ desc)
{
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_list) return;
    WinDesc ds;
    ds.w = win_list[i];
    window_span(ds.w, n_rows, rowptr, ds.s, ds.e);
    ds.nc = ncols[ds.w];
    ds.wp = wptr[ds.w];
    ds.pad = 0;
    desc[i] = ds;
}

hipError_t launch_build_desc(int32_t n_list, const int32_t* win_list, int32_t n_rows, const int32_t* rowptr,
                             const int32_t* ncols, const int64_t* wptr, WinDesc* desc, hipStream_t s)
{
    if (n_list <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_build_desc, dim3((n_list + 255) / 256), dim3(256), 0, s, n_list, win_list, n_rows, rowptr,
                       ncols, wptr, desc);
    return hipGetLastError();
}

// matrix-path launch table: workgroup slices of medium and wide windows
__global__ __launch_bounds__(256) void k_slice_count(int32_t n_list, const int32_t* __restrict__ win_list,
                                                     const int32_t* __restrict__ ncols, int32_t slice_cols,
                                                     int32_t* __restrict__ n_slices, int32_t* __restrict__ f_multi,
                                                     int32_t* __restrict__ n_slots)
{
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_list) return;
    const int32_t nc = ncols[win_list[i]];
    const int32_t ns = (nc + slice_cols - 1) / slice_cols;
    n_slices[i] = ns;
    f_multi[i] = ns > 1 ? 1 : 0;
    n_slots[i] = ns > 1 ? ns : 0;
}

__global__ __launch_bounds__(256) void k_slice_fill(int32_t n_list, const int32_t* __restrict__ win_list,
                                                    const int32_t* __restrict__ ncols, int32_t slice_cols,
                                                    const int64_t* __restrict__ slice_pos,
                                                    const int64_t* __restrict__ multi_pos,
                                                    const int64_t* __restrict__ slot_pos, WgSlice* __restrict__ slices,
                                                    MultiRow* __restrict__ multi)
{
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_list) return;
    const int32_t w = win_list[i];
    const int32_t nc = ncols[w];
    const int32_t ns = (nc + slice_cols - 1) / slice_cols;
    const int32_t slot0 = ns > 1 ? (int32_t)slot_pos[i] : -1;
    for (int32_t q = 0; q < ns; ++q) {
        WgSlice sl;
        sl.w = w;
        sl.kc_begin = q * slice_cols;
        sl.kc_end = min(nc, sl.kc_begin + slice_cols);
        sl.slot = ns > 1 ? slot0 + q : -1;
        slices[slice_pos[i] + q] = sl;
    }
    if (ns > 1) {
        MultiRow m;
        m.row = w; m.first_slot = slot0; m.n_slots = ns; m.pad = 0;
        multi[multi_pos[i]] = m;
    }
}

// per slice and window row: the first non-zero of the row whose condensed column is inside the slice
// (rows with ascending columns only: their condensed columns ascend too)
__global__ __launch_bounds__(256) void k_slice_rows(int32_t n_slices, const WgSlice* __restrict__ slices,
                                                    int32_t n_rows, const int32_t* __restrict__ rowptr,
                                                    const int32_t* __restrict__ erc, int32_t* __restrict__ slice_rows)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n_slices * kH) return;
    const WgSlice sl = slices[t / kH];
    const int64_t row = (int64_t)sl.w * kH + (t % kH);
    int32_t lo = rowptr[min(row, (int64_t)n_rows)], hi = rowptr[min(row + 1, (int64_t)n_rows)];
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if ((erc[mid] >> 4) < sl.kc_begin) lo = mid + 1; else hi = mid;
    }
    slice_rows[t] = lo;
}

hipError_t launch_slice_rows(int32_t n_slices, const WgSlice* slices, int32_t n_rows, const int32_t* rowptr,
                             const int32_t* erc, int32_t* slice_rows, hipStream_t s)
{
    if (n_slices <= 0) return hipSuccess;
    const int64_t n = (int64_t)n_slices * kH;
    hipLaunchKernelGGL(k_slice_rows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n_slices, slices, n_rows,
                       rowptr, erc, slice_rows);
    return hipGetLastError();
}

hipError_t launch_slice_count(int32_t n_list, const int32_t* win_list, const int32_t* ncols, int32_t slice_cols,
                              int32_t* n_slices, int32_t* f_multi, int32_t* n_slots, hipStream_t s)
{
    if (n_list <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_slice_count, dim3((n_list + 255) / 256), dim3(256), 0, s, n_list, win_list, ncols, slice_cols,
                       n_slices, f_multi, n_slots);
    return hipGetLastError();
}

hipError_t launch_slice_fill(int32_t n_list, const int32_t* win_list, const int32_t* ncols, int32_t slice_cols,
                             const int64_t* slice_pos, const int64_t* multi_pos, const int64_t* slot_pos,
                             WgSlice* slices, MultiRow* multi, hipStream_t s)
{
    if (n_list <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_slice_fill, dim3((n_list + 255) / 256), dim3(256), 0, s, n_list, win_list, ncols, slice_cols,
                       slice_pos, multi_pos, slot_pos, slices, multi);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// column panels: panel q of n holds the columns [n_cols*q/n, n_cols*(q+1)/n)
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_panel_split(PanelArgs p)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= p.n_rows) return;
    int32_t lo = p.rowptr[i];
    const int32_t e = p.rowptr[i + 1];
    for (int q = 1; q < p.n_panels; ++q) {
        const int32_t c = (int32_t)((int64_t)p.n_cols * q / p.n_panels);
        int32_t hi = e;
        while (lo < hi) { const int32_t mid = lo + ((hi - lo) >> 1); if (p.colind[mid] < c) lo = mid + 1; else hi = mid; }
        p.split[(int64_t)(q - 1) * p.n_rows + i] = lo;
    }
}

struct PanelRow { int32_t s, e; int is_mid, n_seg; };
__device__ inline PanelRow panel_row(const PanelArgs& p, int q, int64_t i)
{
    PanelRow r{0, 0, 0, 0};
    if (i >= p.n_rows) return r;
    r.s = q == 0 ? p.rowptr[i] : p.split[(int64_t)(q - 1) * p.n_rows + i];
    r.e = q == p.n_panels - 1 ? p.rowptr[i + 1] : p.split[(int64_t)q * p.n_rows + i];
    const int32_t len = r.e - r.s;
    r.n_seg = len > p.long_row ? (len + kSegLen - 1) / kSegLen : 0;
    r.is_mid = r.n_seg == 0 && len > p.mid_row;
    return r;
}

// sums per panel and tile of 1024 rows: mid rows | rows of several segments, segments | partial rows, non-zeros
__global__ __launch_bounds__(256) void k_panel_count(PanelArgs p)
{
    __shared__ unsigned long long smem[12];
    const int tile = blockIdx.x, q = blockIdx.y;
    unsigned long long sum[3] = {0, 0, 0};
    for (int j = 0; j < 4; ++j) {
        const PanelRow r = panel_row(p, q, (int64_t)tile * kTileRows + j * 256 + threadIdx.x);
        sum[0] += (unsigned long long)r.is_mid | (unsigned long long)(r.n_seg > 1) << 32;
        sum[1] += (unsigned long long)r.n_seg | (unsigned long long)(r.n_seg > 1 ? r.n_seg : 0) << 32;
        sum[2] += (unsigned long long)(r.e - r.s);
    }
    block_sums_u64<3>(sum, smem);
    if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < 3; ++i) p.sums[((int64_t)q * p.n_tiles + tile) * 3 + i] = sum[i];
}

__global__ __launch_bounds__(256) void k_panel_fill(PanelArgs p)
{
    __shared__ unsigned long long smem[12];
    const int tile = blockIdx.x, q = blockIdx.y;
    unsigned long long front[3] = {0, 0, 0};
    for_sums<3, false>(p.sums + (int64_t)q * p.n_tiles * 3, p.groups ? p.groups + (int64_t)q * p.n_groups * 3 : nullptr, p.n_tiles, tile, threadIdx.x, 256,
                       [&](const unsigned long long* u, bool) { front[0] += u[0]; front[1] += u[1]; front[2] += u[2]; });
    block_sums_u64<3>(front, smem);
    unsigned long long a = front[0], b = front[1];
    const unsigned long long n = front[2];
    if (tile == p.n_tiles) {                                    // behind the last tile: the totals
        if (threadIdx.x == 0) p.out[q] = PanelTotals{(int64_t)n, (int64_t)(b >> 32), (int32_t)a, (int32_t)b, (int32_t)(a >> 32), 0};
        return;
    }
    for (int j = 0; j < 4; ++j) {
        const int64_t i = (int64_t)tile * kTileRows + j * 256 + threadIdx.x;
        const PanelRow r = panel_row(p, q, i);
        const unsigned long long va = (unsigned long long)r.is_mid | (unsigned long long)(r.n_seg > 1) << 32;
        const unsigned long long vb = (unsigned long long)r.n_seg | (unsigned long long)(r.n_seg > 1 ? r.n_seg : 0) << 32;
        const unsigned long long ea = a + block_scan_u64(va, smem), eb = b + block_scan_u64(vb, smem);
        a += block_sum_u64(va, smem);
        b += block_sum_u64(vb, smem);
        if (r.is_mid) p.mid_rows[q * p.cap_mid + (uint32_t)ea] = (int32_t)i;
        for (int k = 0; k < r.n_seg; ++k)
            p.segs[q * p.cap_segs + (uint32_t)eb + k] = Segment{(int32_t)i, r.s + k * kSegLen, min(r.e, r.s + (k + 1) * kSegLen),
                                                               r.n_seg > 1 ? (int32_t)(eb >> 32) + k : -1};
        if (r.n_seg > 1) p.multi[q * p.cap_multi + (uint32_t)(ea >> 32)] = MultiRow{(int32_t)i, (int32_t)(eb >> 32), r.n_seg, 0};
    }
}

hipError_t launch_panels(const PanelArgs& p_, hipStream_t s)
{
    PanelArgs p = p_;
    p.n_groups = group_count(p.n_tiles);
    p.groups = p.n_groups ? p.sums + 3 * (size_t)p.n_panels * p.n_tiles : nullptr;
    hipLaunchKernelGGL(k_panel_split, dim3((unsigned)(((int64_t)p.n_rows + 255) / 256)), dim3(256), 0, s, p);
    hipLaunchKernelGGL(k_panel_count, dim3((unsigned)p.n_tiles, (unsigned)p.n_panels), dim3(256), 0, s, p);
    if (p.groups) hipLaunchKernelGGL(k_group_sums<3>, dim3((unsigned)p.n_groups, (unsigned)p.n_panels), dim3(256), 0, s, p.n_tiles, p.sums, p.groups);
    hipLaunchKernelGGL(k_panel_fill, dim3((unsigned)p.n_tiles + 1, (unsigned)p.n_panels), dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace hcspmm
