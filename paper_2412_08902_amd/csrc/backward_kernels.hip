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
            if constexpr (VEC) {                                    // (d is a multiple of NT)
                if (n0 + NT * c >= d) continue;
                f32_vec<NT> v;
#pragma unroll
                for (int j = 0; j < NT; ++j) v.v[j] = acc[i][j][r];
                *reinterpret_cast<f32_vec<NT>*>(out + (int64_t)m * d + n0 + NT * c) = v;
            } else {
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    if (n0 + 16 * j + c < d) out[(int64_t)m * d + n0 + 16 * j + c] = acc[i][j][r];
            }
        }
}

// Both products of the backward pass at once, for widths of 65 to 128 either way: dX = S W^T and the spans' parts of
// dW = X^T S.  Apart they read S twice, transpose W in between and take a launch more; together they are bound by the matrix
// units (169,343 x 128 x 128: 11.1 GFLOP, 73 us at the 151 TFLOP/s of a large library product; 65 + 56 + 5 us apart, 111 us here;
// 16,934 rows: 52.8 -> 42.8 us for the whole call).  A workgroup owns a span of 16-row batches as in k_gemm_tn, its two halves of
// four waves taking them in turn (one half alone, a wave per SIMD, waits as much as it multiplies: 120 us).  Per batch a wave adds
// to its MT x NT tiles of dW (2 x 2 waves side by side) and multiplies the 16 rows of S with 32 rows of W.  The batch of S
// comes through LDS, read once and in whole lines: an operand of 16 rows read straight from memory costs the load path 64
// accesses instead of 16, as neighbouring lanes are different rows (133 us).  W stays in LDS; in registers it leaves no room for
// two waves.  A lane's k in step t of unit u is 16u + 4q + t in both operands of dX.
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kGradPitch = 136, kGradPitchW = 132;   // the 16-byte reads of 16 rows, of every other row of W, meet no bank twice
template <int MT, int NT, int K16>
__global__ __launch_bounds__(512, 2) void k_gemm_grad(int64_t n_rows, const float* __restrict__ X, int64_t ldx, int32_t d_in,
                                                      const float* __restrict__ S, int64_t lds_, int32_t d,
                                                      const float* __restrict__ W, int64_t ldw, float* __restrict__ dX, int64_t lddx,
                                                      int vec, float* __restrict__ partial)
{
    const int half = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), tid = threadIdx.x & 255;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = threadIdx.x & 63, c = lane & 15, q = lane >> 4;
    const int m0 = wave / 2 * 16 * MT, n0 = wave % 2 * 16 * NT;     // this wave's tiles of dW
    extern __shared__ __attribute__((aligned(16))) float smem[];   // two tiles of S per half; the second half's sums at the end
    float* __restrict__ tile = smem + half * 2 * 16 * kGradPitch;
    const int xo = min(m0 + MT * c, d_in - MT);
    const int i0 = wave * 32 + 2 * c;                               // this lane's two columns of dX
    // W stays in LDS, rows past it and columns past S zero
    float* __restrict__ wt = smem + 4 * 16 * kGradPitch;
    const float* __restrict__ cw = wt + i0 * kGradPitchW + 4 * q;
    v4f_bw acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (v4f_bw){0.f, 0.f, 0.f, 0.f};
    constexpr int PIECES = 16 * 4 * K16, ITERS = (PIECES + 255) / 256;      // pieces of four of a batch of S, per thread
    int sr[ITERS], sk[ITERS];
#pragma unroll
    for (int i = 0; i < ITERS; ++i) {
        const int at = tid + 256 * i;
        sr[i] = at / (4 * K16);
        sk[i] = at % (4 * K16) * 4;
    }
    f4_any next[ITERS];
    auto request_s = [&](int64_t r0) {
#pragma unroll
        for (int i = 0; i < ITERS; ++i)
            if (PIECES % 256 == 0 || sr[i] < 16)
                next[i] = *reinterpret_cast<const f4_any*>(S + min(r0 + sr[i], n_rows - 1) * lds_ + (sk[i] < d ? sk[i] : 0));
    };
    // rows past the matrix and columns past S are zeros
    auto park = [&](int64_t r0, float* __restrict__ to) {
#pragma unroll
        for (int i = 0; i < ITERS; ++i) {
            if (PIECES % 256 != 0 && sr[i] >= 16) continue;
            const bool in = sk[i] < d && r0 + sr[i] < n_rows;
            *reinterpret_cast<float4*>(to + sr[i] * kGradPitch + sk[i]) =
                make_float4(in ? next[i].x : 0.f, in ? next[i].y : 0.f, in ? next[i].z : 0.f, in ? next[i].w : 0.f);
        }
    };
    f32_vec<MT> x[4];
    auto request_x = [&](int64_t r0, int t) { x[t] = *reinterpret_cast<const f32_vec<MT>*>(X + min(r0 + 4 * t + q, n_rows - 1) * ldx + xo); };
    const uint32_t xl = (uint32_t)q * (uint32_t)ldx * 4u + (uint32_t)xo * 4u;    // (16 rows of X reach less than 4 GiB: gemm_grad_usable)
    const int64_t batches = (n_rows + 15) / 16, G = gridDim.x, b_begin = blockIdx.x * batches / G, b_end = (blockIdx.x + 1) * batches / G;
    const int64_t last = b_end - 1;
    if (b_begin + half < b_end) {
        const int64_t r0 = (b_begin + half) * 16;
        request_s(r0);
#pragma unroll
        for (int t = 0; t < 4; ++t) request_x(r0, t);
    }
    {
        f4_any v[K16];
#pragma unroll
        for (int i = 0; i < K16; ++i) {
            const int at = (int)threadIdx.x + 512 * i, row = at / (4 * K16), col = at % (4 * K16) * 4;
            v[i] = *reinterpret_cast<const f4_any*>(W + (int64_t)(row < d_in && col < d ? row : 0) * ldw + (row < d_in && col < d ? col : 0));
        }
#pragma unroll
        for (int i = 0; i < K16; ++i) {
            const int at = (int)threadIdx.x + 512 * i, row = at / (4 * K16), col = at % (4 * K16) * 4;
            const bool in = row < d_in && col < d;
            *reinterpret_cast<float4*>(wt + row * kGradPitchW + col) = make_float4(in ? v[i].x : 0.f, in ? v[i].y : 0.f, in ? v[i].z : 0.f, in ? v[i].w : 0.f);
        }
    }
    if (b_begin + half < b_end) park((b_begin + half) * 16, tile);
    __syncthreads();
    int turn = 0;
    for (int64_t b = b_begin + half; b - half < b_end; b += 2, turn ^= 1) {
        if (b >= b_end) { __syncthreads(); break; }                 // (the second half's last turn; uniform in the half)
        const float* __restrict__ cur = tile + turn * 16 * kGradPitch;
        const int64_t r0 = b * 16, r1 = min(b + 2, last) * 16;
        if (r0 + 16 > n_rows) {                                     // rows past the matrix (the last batch; uniform)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (r0 + 4 * t + q >= n_rows) {
#pragma unroll
                    for (int i = 0; i < MT; ++i) x[t].v[i] = 0.f;
                }
        }
        request_s(r1);
        __builtin_amdgcn_sched_barrier(0);
        v4f_bw dx[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        // (operands from LDS a few steps ahead, in this order: left alone the compiler reads each right before its products)
        const float* __restrict__ ca = cur + c * kGradPitch + 4 * q;
        const float* __restrict__ cy = cur + q * kGradPitch + n0 + NT * c;
        float4 a[2], w[2][2];
        f32_vec<NT> y[2];
        auto read = [&](int u) {
            a[u & 1] = *reinterpret_cast<const float4*>(ca + 16 * u);
            w[u & 1][0] = *reinterpret_cast<const float4*>(cw + 16 * u);
            w[u & 1][1] = *reinterpret_cast<const float4*>(cw + kGradPitchW + 16 * u);
        };
        auto read_y = [&](int t) { y[t & 1] = *reinterpret_cast<const f32_vec<NT>*>(cy + 4 * t * kGradPitch); };
        read(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < K16; ++u) {
            if (u + 1 < K16) read(u + 1);
            else read_y(0);
            __builtin_amdgcn_sched_barrier(0);
            const float av[4] = {a[u & 1].x, a[u & 1].y, a[u & 1].z, a[u & 1].w};
            const float w0[4] = {w[u & 1][0].x, w[u & 1][0].y, w[u & 1][0].z, w[u & 1][0].w};
            const float w1[4] = {w[u & 1][1].x, w[u & 1][1].y, w[u & 1][1].z, w[u & 1][1].w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                dx[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t], w0[t], dx[0], 0, 0, 0);
                dx[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t], w1[t], dx[1], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const char* __restrict__ xb = reinterpret_cast<const char*>(X + r1 * ldx);
        uint32_t xo_t[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) xo_t[t] = xl + (uint32_t)(4 * t) * (uint32_t)ldx * 4u;
        if (r1 + 16 > n_rows) {                                     // (uniform) rows past the matrix repeat its last one
#pragma unroll
            for (int t = 0; t < 4; ++t) xo_t[t] = (uint32_t)min((int64_t)(4 * t + q), n_rows - 1 - r1) * (uint32_t)ldx * 4u + (uint32_t)xo * 4u;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (t + 1 < 4) read_y(t + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t].v[i], y[t & 1].v[j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            x[t] = *reinterpret_cast<const f32_vec<MT>*>(xb + xo_t[t]);
            __builtin_amdgcn_sched_barrier(0);
        }
        park(r1, tile + (turn ^ 1) * 16 * kGradPitch);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t row = r0 + 4 * q + r;
            if (row >= n_rows) continue;
            float* __restrict__ p = dX + row * lddx + i0;
            if (vec && i0 + 1 < d_in) {
                *reinterpret_cast<float2*>(p) = make_float2(dx[0][r], dx[1][r]);
            } else {
                if (i0 < d_in) p[0] = dx[0][r];
                if (i0 + 1 < d_in) p[1] = dx[1][r];
            }
        }
        __syncthreads();                                            // the next tile is in place, and nobody reads this one
    }
    // the second half's sums are added to the first's
    __syncthreads();
    if (half) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) *reinterpret_cast<v4f_bw*>(smem + (((wave * MT + i) * NT + j) * 64 + lane) * 4) = acc[i][j];
    }
    __syncthreads();
    if (half || m0 >= d_in || n0 >= d) return;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] += *reinterpret_cast<const v4f_bw*>(smem + (((wave * MT + i) * NT + j) * 64 + lane) * 4);
    float* __restrict__ out = partial + (int64_t)blockIdx.x * d_in * d;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + MT * (4 * q + r) + i;
            if (m >= d_in || n0 + NT * c >= d) continue;            // (d is a multiple of NT)
            f32_vec<NT> v;
#pragma unroll
            for (int j = 0; j < NT; ++j) v.v[j] = acc[i][j][r];
            *reinterpret_cast<f32_vec<NT>*>(out + (int64_t)m * d + n0 + NT * c) = v;
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

// Whether launch_gemm_grad takes these products: four waves' tiles of dW as k_gemm_tn cuts them (so that the partial products
// have the room they need), whole vectors of their columns, S's rows in whole pieces of four.  The four waves multiply 128
// columns of dX whatever d_in is, which shows where the product is large (apart / together, us: 169,343 rows, d_in 128, d 128: 285 /
// 272, 112, 72: 207 / 197, 96, 96: 214 / 211, 96, 128: 258 / 260, 72, 128: 251 / 257; 40,000 rows, 96, 96: 58 / 53).
bool gemm_grad_usable(int64_t n_rows, int64_t ldx, int32_t d_in, int32_t d)
{
    if (ldx >= (1 << 26) || (d_in <= 96 && n_rows >= 65536) || d_in <= 64 || d_in > 128 || d <= 64 || d > 128 || d % 4 != 0) return false;
    const TnShape t = tn_shape(n_rows, d_in, d);
    return t.qm == 2 && t.qn == 2 && t.ny == 1 && t.nz == 1 && d_in % t.mt == 0 && d % t.nt == 0;
}

// dX (n_rows x d_in) = S W^T and dW as launch_gemm_tn
hipError_t launch_gemm_grad(int64_t n_rows, const float* X, int64_t ldx, int32_t d_in, const float* S, int64_t lds_, int32_t d,
                            const float* W, int64_t ldw, float* dX, int64_t lddx, float* dW, int64_t lddw, float* partial, hipStream_t s)
{
    if (!gemm_grad_usable(n_rows, ldx, d_in, d)) return hipErrorInvalidValue;
    const TnShape t = tn_shape(n_rows, d_in, d);
    const int vec = lddx % 2 == 0 && (uintptr_t)dX % 8 == 0;
    constexpr size_t kLds = (4 * 16 * kGradPitch + 128 * kGradPitchW) * sizeof(float);   // 102 KB; the second half's sums, 64 KB at most, lie over it
#define HC_GRAD(MT, NT, KK)                                                                                    \
    {                                                                                                          \
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_grad<MT, NT, KK>), \
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);                                            \
        if (attr != hipSuccess) return attr;                                                                   \
    }                                                                                                          \
    hipLaunchKernelGGL((k_gemm_grad<MT, NT, KK>), dim3((unsigned)t.spans), dim3(512), kLds, s, n_rows, X, ldx, d_in, S, lds_, d, W, ldw, dX, lddx, vec, partial)
#define HC_GRAD_K(MT) switch ((d + 15) / 16) { case 5: { HC_GRAD(MT, 3, 5); } break; case 6: { HC_GRAD(MT, 3, 6); } break; case 7: { HC_GRAD(MT, 4, 7); } break; default: { HC_GRAD(MT, 4, 8); } break; }
    if (t.mt == 3) HC_GRAD_K(3)
    else HC_GRAD_K(4)
#undef HC_GRAD_K
#undef HC_GRAD
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t count = (int64_t)d_in * d;
    hipLaunchKernelGGL(k_sum_partials, dim3((unsigned)((count + 15) / 16)), dim3(256), 0, s, t.spans, count, d, partial, dW, lddw);
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
