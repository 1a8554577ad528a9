// Dense pieces of the layer's backward pass (Eq. 3): the weight gradient dW = X^T S, a reduction
// over all rows of the graph, plus the two small helpers around it (activation mask on the incoming
// gradient, transpose of W for the product S W^T that the update epilogue computes).
//
// dW = X^T S is a product with a short output (d_in x d) and a contraction as long as the graph has rows: reading X and S
// once and the matrix units (v_mfma_f32_16x16x4_f32) bound it about equally at 128 x 128.  Both operands of a step of four
// rows are rows as they lie in memory -- lane (c = l%16, q = l/16) supplies A(column, k = q) = X[row q][..] and B(k = q,
// column) = S[row q][..] -- so they are loaded straight into registers: a wave owns up to 4 x 4 tiles of 16 x 16 outputs
// (tile i of MT holds the columns base + MT*c + i, so MT values are one vector load; or base + 16*i + c, one value each,
// where the width is no multiple of MT), keeps a ring of four steps in flight and never meets a barrier before its end.
// A workgroup's waves are Q such blocks times RG row groups; the row groups' sums are added through LDS, every workgroup
// (one per CU) writes one partial product and a second kernel adds the partials, all in an order that depends on sizes only.
// (64-row stages through LDS with two barriers each, 512 partial products: 169,343 x 128 x 128 took 106 us + 8 us,
// now 61 us + 6 us.)
#include "common.hpp"

namespace hcspmm {

typedef float v4f_bw __attribute__((ext_vector_type(4)));
template <int N> struct __attribute__((packed, aligned(4))) f32_vec { float v[N]; };

constexpr int kTnSteps = 4, kTnBatch = 4 * kTnSteps;                // steps and rows per batch
constexpr int kTnWaves = 8;                                         // waves per workgroup at most

// How a d_in x d output is cut: MT x NT tiles per wave, qm x qn waves side by side in a workgroup, ny x nz workgroups, rg row
// groups per workgroup, `spans` workgroups along the rows.
struct TnShape { int mt, nt, qm, qn, ny, nz, rg; int32_t spans; };
static TnShape tn_shape(int64_t n_rows, int32_t d_in, int32_t d)
{
    TnShape t;
    const int m16 = (d_in + 15) / 16, n16 = (d + 15) / 16;
    const int qm_all = (m16 + 3) / 4, qn_all = (n16 + 3) / 4;
    t.mt = (m16 + qm_all - 1) / qm_all;
    t.nt = (n16 + qn_all - 1) / qn_all;
    // One wave per SIMD where it has more than eight tiles (a step's products take four times as long as its loads then, and
    // more waves only cost start-up, reduction and larger outputs per workgroup: 60,000 x 256 x 256: 16 waves 115 us, 8 waves
    // 90 us, 4 waves 80 us; 169,343 x 128 x 128: 82, 77, 74 us), two for smaller blocks, which are bound by their loads
    // (400,000 x 32 x 128: 4 waves 56.7 us, 8 waves 54.3 us).
    const int waves = t.mt * t.nt > 8 ? 4 : kTnWaves;
    t.nz = (qn_all + waves - 1) / waves;
    t.qn = (qn_all + t.nz - 1) / t.nz;
    const int most = waves / t.qn;
    t.ny = (qm_all + most - 1) / most;
    t.qm = (qm_all + t.ny - 1) / t.ny;
    // row groups: the four SIMDs of a CU should carry equally many waves, and as many as fit
    const int q = t.qm * t.qn;
    t.rg = 1;
    double best = 0.0;
    for (int rg = 1; rg * q <= waves; ++rg) {
        const double even = (double)(rg * q) / ((rg * q + 3) / 4 * 4);
        if (even >= best) { best = even; t.rg = rg; }
    }
    const int64_t batches = (n_rows + kTnBatch - 1) / kTnBatch;
    int64_t spans = 256 / ((int64_t)t.ny * t.nz);                   // a workgroup per CU
    if (spans > batches / (2 * t.rg)) spans = batches / (2 * t.rg); // two batches per wave at least
    t.spans = (int32_t)(spans < 1 ? 1 : spans);
    return t;
}

template <int MT, int NT, bool VEC>
__global__ __launch_bounds__(64 * kTnWaves) void k_gemm_tn(int64_t n_rows, const float* __restrict__ X, int64_t ldx, int32_t d_in,
                                                           const float* __restrict__ S, int64_t lds_, int32_t d, int qm, int qn,
                                                           int rg_count, float* __restrict__ partial)
{
    extern __shared__ float red[];                                  // rg_count / 2 * qm * qn blocks of 64 x 4*MT*NT sums
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 15, q = lane >> 4;
    const int blocks = qm * qn, rg = wave / blocks, blk = wave % blocks;
    const int m0 = ((int)blockIdx.y * qm + blk / qn) * 16 * MT, n0 = ((int)blockIdx.z * qn + blk % qn) * 16 * NT;
    const bool live = m0 < d_in && n0 < d;                          // (uniform; a block of the last y or z may be all padding)
    // column offsets of this lane's values inside a row; past the matrix they repeat its last columns (and are not stored)
    int xo[VEC ? 1 : MT], so[VEC ? 1 : NT];
    if constexpr (VEC) {
        xo[0] = min(m0 + MT * c, d_in - MT);
        so[0] = min(n0 + NT * c, d - NT);
    } else {
#pragma unroll
        for (int i = 0; i < MT; ++i) xo[i] = min(m0 + 16 * i + c, d_in - 1);
#pragma unroll
        for (int j = 0; j < NT; ++j) so[j] = min(n0 + 16 * j + c, d - 1);
    }
    v4f_bw acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (v4f_bw){0.f, 0.f, 0.f, 0.f};
    constexpr int RING = 4;                                         // steps in flight
    float x[RING][MT], y[RING][NT];
    auto fetch = [&](int64_t r0 /* uniform */, int dr, float (&a)[MT], float (&b)[NT]) {
        const float* __restrict__ px = X + r0 * ldx + dr * ldx;
        const float* __restrict__ ps = S + r0 * lds_ + dr * lds_;
        if constexpr (VEC) {
            const f32_vec<MT> va = *reinterpret_cast<const f32_vec<MT>*>(px + xo[0]);
            const f32_vec<NT> vb = *reinterpret_cast<const f32_vec<NT>*>(ps + so[0]);
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = va.v[i];
#pragma unroll
            for (int j = 0; j < NT; ++j) b[j] = vb.v[j];
        } else {
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = px[xo[i]];
#pragma unroll
            for (int j = 0; j < NT; ++j) b[j] = ps[so[j]];
        }
    };
    auto multiply = [&](const float (&a)[MT], const float (&b)[NT]) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    };
    // the workgroup's whole batches, taken in turn by its row groups (each reads a stretch of its own close to the others')
    const int64_t whole = n_rows / kTnBatch, G = gridDim.x;
    const int64_t b_end = (blockIdx.x + 1) * whole / G;
    int64_t b = blockIdx.x * whole / G + rg;
    if (live && b < b_end) {
        const int64_t last = b_end - 1;
        // row of step u of batch b; requests past the span repeat its last batch (branches would cost waits at their joins)
        auto row = [&](int64_t bb, int u) { return min(bb, last) * kTnBatch + 4 * u; };
#pragma unroll
        for (int u = 0; u < RING; ++u) {
            fetch(row(b, u), q, x[u], y[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (; b < b_end; b += rg_count) {
#pragma unroll
            for (int u = 0; u < kTnSteps; ++u) {
                multiply(x[u % RING], y[u % RING]);
                __builtin_amdgcn_sched_barrier(0);
                fetch(u + RING < kTnSteps ? row(b, u + RING) : row(b + rg_count, u + RING - kTnSteps), q, x[u % RING], y[u % RING]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // the last rows of the matrix, fewer than a batch: the last workgroup's first row group, zero-filled
    if (live && rg == 0 && blockIdx.x == gridDim.x - 1) {
        for (int64_t r0 = whole * kTnBatch; r0 < n_rows; r0 += 4) {
            fetch(r0, (int)min((int64_t)q, n_rows - 1 - r0), x[0], y[0]);
            if (r0 + q >= n_rows) {
#pragma unroll
                for (int i = 0; i < MT; ++i) x[0][i] = 0.f;
#pragma unroll
                for (int j = 0; j < NT; ++j) y[0][j] = 0.f;
            }
            multiply(x[0], y[0]);
        }
    }
    // add the row groups: the upper half's sums go through LDS to the lower half, until one is left
    for (int n = rg_count; n > 1;) {
        const int half = (n + 1) / 2;
        if (rg >= half && rg < n) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    *reinterpret_cast<v4f_bw*>(red + ((((rg - half) * blocks + blk) * MT * NT + i * NT + j) * 64 + lane) * 4) = acc[i][j];
        }
        __syncthreads();
        if (rg + half < n) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] += *reinterpret_cast<const v4f_bw*>(red + (((rg * blocks + blk) * MT * NT + i * NT + j) * 64 + lane) * 4);
        }
        __syncthreads();
        n = half;
    }
    if (rg != 0 || !live) return;
    // partial[span][m][n]; register r of lane (c, q) in tile (i, j) is the output of X's column 4q + r and S's column c there
    float* __restrict__ out = partial + (int64_t)blockIdx.x * d_in * d;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = VEC ? m0 + MT * (4 * q + r) + i : m0 + 16 * i + 4 * q + r;
            if (m >= d_in) continue;
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int n = VEC ? n0 + NT * c + j : n0 + 16 * j + c;
                if (n < d) out[(int64_t)m * d + n] = acc[i][j][r];
            }
        }
}

// out[e] = sum over spans of partial[span][e], in an order that depends only on the span count: 16
// threads per output each add every 16th span in ascending order, then one of them adds the 16 sums
// in ascending order.
__global__ __launch_bounds__(256) void k_sum_partials(int32_t n_spans, int64_t count, int32_t d,
                                                      const float* __restrict__ partial, float* __restrict__ out,
                                                      int64_t ldo)
{
    __shared__ float red[16][17];
    const int o = threadIdx.x & 15, j = threadIdx.x >> 4;
    const int64_t e = (int64_t)blockIdx.x * 16 + o;
    float s = 0.f;
    if (e < count) {
#pragma unroll 16
        for (int32_t p = j; p < n_spans; p += 16) s += partial[(int64_t)p * count + e];
    }
    red[j][o] = s;
    __syncthreads();
    if (j == 0 && e < count) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += red[k][o];
        out[(e / d) * ldo + e % d] = t;
    }
}

int32_t gemm_tn_spans(int64_t n_rows, int32_t d_in, int32_t d) { return tn_shape(n_rows, d_in, d).spans; }

// dW (d_in x d, pitch lddw) = X^T S for X n_rows x d_in and S n_rows x d; partial holds
// gemm_tn_spans(n_rows, d_in, d) * d_in * d floats.
hipError_t launch_gemm_tn(int64_t n_rows, const float* X, int64_t ldx, int32_t d_in, const float* S, int64_t lds_,
                          int32_t d, float* dW, int64_t lddw, float* partial, hipStream_t s)
{
    const TnShape t = tn_shape(n_rows, d_in, d);
    const dim3 grid((unsigned)t.spans, (unsigned)t.ny, (unsigned)t.nz), block(64 * t.qm * t.qn * t.rg);
    const size_t lds_bytes = (size_t)(t.rg / 2) * t.qm * t.qn * 64 * 4 * t.mt * t.nt * sizeof(float);      // 64 KB at most
    const bool vec = d_in % t.mt == 0 && d % t.nt == 0;
    hipError_t e = hipSuccess;
#define HC_TN(MT, NT, V)                                                                                       \
    {                                                                                                          \
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_tn<MT, NT, V>), \
            hipFuncAttributeMaxDynamicSharedMemorySize, kTnWaves / 2 * 64 * 4 * MT * NT * (int)sizeof(float)); \
        if (attr != hipSuccess) return attr;     /* (once per process: later calls may run under stream capture) */ \
        hipLaunchKernelGGL((k_gemm_tn<MT, NT, V>), grid, block, lds_bytes, s, n_rows, X, ldx, d_in, S, lds_, d, t.qm, t.qn, t.rg, partial); \
    }
#define HC_TN_V(MT, NT) if (vec) HC_TN(MT, NT, true) else HC_TN(MT, NT, false) break
#define HC_TN_N(MT) switch (t.nt) { case 1: HC_TN_V(MT, 1); case 2: HC_TN_V(MT, 2); case 3: HC_TN_V(MT, 3); default: HC_TN_V(MT, 4); } break
    switch (t.mt) { case 1: HC_TN_N(1); case 2: HC_TN_N(2); case 3: HC_TN_N(3); default: HC_TN_N(4); }
#undef HC_TN_N
#undef HC_TN_V
#undef HC_TN
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int64_t count = (int64_t)d_in * d;
    hipLaunchKernelGGL(k_sum_partials, dim3((unsigned)((count + 15) / 16)), dim3(256), 0, s, t.spans, count, d, partial,
                       dW, lddw);
    return hipGetLastError();
}

// Gm = G where the forward output is positive, else 0 (derivative of max(0, .)); Gm is n x d, pitch ldo (it may be G
// itself).  VEC = 4: d and all pitches are multiples of 4 and the bases 16-byte aligned.
template <int VEC>
__global__ __launch_bounds__(256) void k_relu_mask(int64_t n, int32_t d, const float* G, int64_t ldg,
                                                   const float* __restrict__ Yf, int64_t ldy, float* Gm, int64_t ldo)
{
    const int per_row = d / VEC;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n * per_row) return;
    const int64_t r = e / per_row;
    const int c = (int)(e % per_row) * VEC;
    if constexpr (VEC == 4) {
        const float4 g = *reinterpret_cast<const float4*>(G + r * ldg + c);
        const float4 y = *reinterpret_cast<const float4*>(Yf + r * ldy + c);
        *reinterpret_cast<float4*>(Gm + r * ldo + c) =
            make_float4(y.x > 0.f ? g.x : 0.f, y.y > 0.f ? g.y : 0.f, y.z > 0.f ? g.z : 0.f, y.w > 0.f ? g.w : 0.f);
    } else {
        Gm[r * ldo + c] = Yf[r * ldy + c] > 0.f ? G[r * ldg + c] : 0.f;
    }
}

hipError_t launch_relu_mask(int64_t n, int32_t d, const float* G, int64_t ldg, const float* Yf, int64_t ldy, float* Gm,
                            int64_t ldo, hipStream_t s)
{
    if (n <= 0 || d <= 0) return hipSuccess;
    const bool vec = d % 4 == 0 && ldg % 4 == 0 && ldy % 4 == 0 && ldo % 4 == 0 && (uintptr_t)G % 16 == 0 &&
                     (uintptr_t)Yf % 16 == 0 && (uintptr_t)Gm % 16 == 0;
    const int64_t count = n * (vec ? d / 4 : d);
    const dim3 grid((unsigned)((count + 255) / 256));
    if (vec) hipLaunchKernelGGL(k_relu_mask<4>, grid, dim3(256), 0, s, n, d, G, ldg, Yf, ldy, Gm, ldo);
    else hipLaunchKernelGGL(k_relu_mask<1>, grid, dim3(256), 0, s, n, d, G, ldg, Yf, ldy, Gm, ldo);
    return hipGetLastError();
}

// Wt (cols x rows, pitch rows) = transpose of W (rows x cols, pitch ldw); W is small
__global__ __launch_bounds__(256) void k_transpose(int32_t rows, int32_t cols, const float* __restrict__ W, int64_t ldw,
                                                   float* __restrict__ Wt)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)rows * cols) return;
    const int64_t c = e / rows, r = e % rows;
    Wt[e] = W[r * ldw + c];
}

hipError_t launch_transpose(int32_t rows, int32_t cols, const float* W, int64_t ldw, float* Wt, hipStream_t s)
{
    const int64_t count = (int64_t)rows * cols;
    hipLaunchKernelGGL(k_transpose, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, rows, cols, W, ldw, Wt);
    return hipGetLastError();
}

}  // namespace hcspmm
