// Scalar path: SpMM straight from CSR for the windows the selector leaves on the vector ALUs
// (Alg. 1 gives the arithmetic, Alg. 3 the mapping idea: a group of lanes owns one output row and
// each lane one slice of the dense width, so X rows are read as whole contiguous segments).
//
// wave64 mapping: a group of 16 lanes -- one DPP row -- owns an output row, every lane holds NV
// vectors of VEC consecutive columns; a wave works on four rows (short rows) or on four non-zeros
// of the same row (mid and long rows) per load instruction.  (Other forms for narrow rows: Gather.)  Column indices and values are fetched
// 16 at a time with one coalesced load per group and handed round by DPP row broadcasts, which are
// operands of the address add and of the multiply-adds themselves: per non-zero and group one add,
// NV loads and NV*VEC multiply-adds, nothing else.  (Handing them round through LDS, 64-bit row
// addresses and 8-lane groups used to cost ~30 issue slots per load and 86 registers: a pass over
// 115 M non-zeros took 0.76 ms with rows of 16 BYTES, i.e. with next to nothing to gather.)  Row
// addresses are a uniform base plus a 32-bit byte offset; matrices X of 4 GiB and more take the
// WIDE form with 64-bit row offsets.  X is read directly from global memory / L2 (the paper found
// staging X in shared memory a loss on this path).  Three tiers by row length balance power-law
// degree distributions:
//   short rows  a lane group owns a row (or takes a few consecutive ones, on matrices whose launch
//               would not fit otherwise: csr_grid.hpp), and the workgroups
//               reach the XCDs in runs so that neighbouring rows share an L2;
//   mid rows    one wave per row, the groups stride over the row and combine with cross-lane adds;
//   long rows   one workgroup per segment of kSegLen non-zeros, combined through LDS in a fixed
//               order (and, for rows of several segments, through partial rows in memory).
// Wide X may be cut into column slices that different XCDs own (see k_csr).
#include <cstdlib>
#include <utility>

#include "common.hpp"
#include "csr_grid.hpp"
#include "update_tile.hpp"

namespace hcspmm {

template <int VEC> __device__ inline void vzero(float (&a)[VEC])
{
#pragma unroll
    for (int i = 0; i < VEC; ++i) a[i] = 0.f;
}

template <int N, class F, int... I> __device__ __forceinline__ void unrolled_impl(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void unrolled(F&& f) { unrolled_impl<N>(f, std::make_integer_sequence<int, N>{}); }

// lane I of the 16-lane row, in every lane of the row (a DPP operand: no instruction of its own where the user allows one)
template <int I> __device__ __forceinline__ uint32_t row_bcast(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + I, 0xf, 0xf, true);
}
template <int I> __device__ __forceinline__ float row_bcast(float x) { return __uint_as_float(row_bcast<I>(__float_as_uint(x))); }

// ---- launch description ---------------------------------------------------------------------
// Workgroups are numbered heaviest first: long-row segments, then mid rows (four per workgroup),
// then the blocks of short rows, so the short rows fill the machine while the last long rows
// drain instead of each tier waiting for the previous one's tail.
struct CsrWork {
    int32_t n_segs;
    const Segment* segs;
    float* partial;
    int32_t n_mid;
    const int32_t* mid_rows;
    int32_t n_items;
    const int32_t* row_list;
    const uint8_t* route;
    int32_t mid_row;            // longest row of the short tier, or of the mid tier when that has no list (a matrix of few rows)
    CsrGrid grid;               // (right behind mid_row: one load brings what a short row's workgroup needs)
    int32_t y_vec;              // Y rows allow vector stores
    int32_t skip_empty;         // a row without non-zeros changes nothing (a column panel that adds to Y)
};

// One gathered vector as it sits in registers (16-bit elements stay packed until they are multiplied).  Loads are
// aligned to 4 bytes at least (2 for single 16-bit elements), which is all the hardware asks for.
typedef uint32_t raw4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t raw2 __attribute__((ext_vector_type(2), aligned(4)));
template <int BYTES> struct Raw { uint32_t w[BYTES / 4]; };
template <> struct Raw<2> { uint32_t w[1]; };
template <int BYTES> __device__ __forceinline__ void raw_load(const char* __restrict__ p, Raw<BYTES>& r)
{
    static_assert(BYTES == 2 || BYTES == 4 || BYTES == 8 || BYTES == 16, "vector sizes");
    if constexpr (BYTES == 16) { const raw4 v = *reinterpret_cast<const raw4*>(p); r.w[0] = v.x; r.w[1] = v.y; r.w[2] = v.z; r.w[3] = v.w; }
    else if constexpr (BYTES == 8) { const raw2 v = *reinterpret_cast<const raw2*>(p); r.w[0] = v.x; r.w[1] = v.y; }
    else if constexpr (BYTES == 4) { r.w[0] = *reinterpret_cast<const uint32_t*>(p); }
    else { r.w[0] = *reinterpret_cast<const unsigned short*>(p); }
}

// VEC consecutive floats at any 4-byte aligned place
template <int VEC> struct __attribute__((packed, aligned(4))) f32_any { float v[VEC]; };

// XK: element kind of X -- 0 fp32, 1 bf16, 2 fp16.  16-bit elements are widened to fp32; all arithmetic is fp32.
template <int XK> __device__ __forceinline__ float widened(const uint32_t* w, int i)
{
    if constexpr (XK == 0) return __uint_as_float(w[i]);
    else if constexpr (XK == 1) return __uint_as_float((i & 1) ? (w[i >> 1] & 0xffff0000u) : (w[i >> 1] << 16));
    else return (float)__builtin_bit_cast(_Float16, (unsigned short)((i & 1) ? (w[i >> 1] >> 16) : (w[i >> 1] & 0xffffu)));
}

// The gather of one lane group: GROUP lanes own an output row, LANES of them read a row of X, NV vectors of VEC elements each:
// COLS columns of an X row in all.  Three forms:
//   16 of 16   one non-zero at a time;
//   8 of 16    the two halves of the group work on two non-zeros at a time (slots 2t and 2t+1) and are added when the row is
//              done.  A vector-memory instruction takes the CU's load path 16 clocks whether its lanes ask for 8 or 16 bytes
//              (measured on cache hits: 140 G rows of 128 bytes per second with 16 lanes x 8 bytes, 206 G with 8 x 16), so
//              rows of up to 128 bytes are read by 8 lanes; the second broadcast that this takes is free, the VALU has slack;
//   8 of 8     a half of the 16 DPP lanes owns a row of its own.  Twice the output rows per wave: where rows are short and
//              narrow a launch is bound by how fast waves start and drain (see narrow_rows).
// PANEL: a column panel's share of the rows -- each row's end is read from a.rowend, and results may be added to rows of fp32
// sums.  (Kept out of the plain kernels, which have no scalar register to spare in 128-byte rows: power law, fp32, 32
// columns, 39.7 -> 35.1 us.)
// MASK: elements of X count where a.x_mask has their bit.  A lane of the group asks for the 64 bits of its non-zero's row and 64 columns,
// once per 16 non-zeros and ahead of their X rows; the words are handed round like indices and values.
template <int XK, int VEC, int NV, int LANES_, int GROUP_, bool WIDE, bool PANEL = false, bool MASK = false> struct Gather {
    static_assert(!MASK || (XK == 0 && VEC == 4 && LANES_ == 16 && GROUP_ == 16 && !WIDE && !PANEL), "forms with a mask");
    static constexpr bool MANY = WIDE;                          // several rows to a group
    static constexpr int LANES = LANES_, GROUP = GROUP_, SPLIT = GROUP / LANES, STEPS = GROUP / SPLIT;
    static_assert((GROUP == 16 && (LANES == 16 || LANES == 8)) || (GROUP == 8 && LANES == 8), "forms");
    static constexpr int ES = XK == 0 ? 4 : 2;
    static constexpr int BYTES = VEC * ES;
    static constexpr int COLS = LANES * VEC * NV;
    static constexpr int N = VEC * NV;                          // columns per lane
    static constexpr int WORDS = (BYTES < 4 ? 1 : BYTES / 4) * NV;
    static constexpr int U = SPLIT == 2 ? 4 : WORDS <= 4 ? 8 : (WORDS <= 8 ? 4 : 2);   // rows requested before the first is used
    static constexpr int RAW = BYTES;
    // Waves per SIMD the registers are held to.  Short rows are bound by their chain of dependent loads, so 16-byte
    // vectors with one accumulator set are squeezed into 64 registers for all 8 waves (community graph, bf16, 64 columns:
    // 37.0 -> 32.2 us), in fp32 into 72 for 7: the whole batch of steps() spills at 64 (2.4 M rows of 51, 32 columns: 2102 us
    // with 7 waves, 2122 with 8 and half a batch in flight, 2234 with 8 and the spill); wider rows are bound by the traffic
    // behind L2 and lose more to the squeeze (fp32, 128 columns: 120.8 -> 137 us).
    static constexpr int WAVES = LANES == 8 ? (XK == 0 ? 7 : 8) : (XK != 0 && VEC == 8 && NV == 1) ? 6 : 1;

    const char* X;              // uniform: first column of the slice
    uint64_t ldxb;              // bytes between rows (uniform)
    uint32_t lane_off[NV];      // byte offset of this lane's vectors inside the slice
    int shift[NV];              // leading elements of a vector that belong to the lane to the left
    bool ok[NV];                // the vector has columns of the slice
    const char* bits;           // MASK: the slice's first 64 columns of the mask (uniform), bytes to the next 64, this lane's first bit
    size_t next_bits;
    int bit;

    // columns [c0, c0 + w) of X, w <= COLS; a vector that would stick out of the row is moved left so that it ends at the
    // row's last column of the slice (the elements it then shares with its left neighbour are not stored)
    __device__ __forceinline__ void init(const SpmmArgs& a, int c0, int w, int lig_)
    {
        const int lig = lig_ % LANES;
        X = static_cast<const char*>(a.X);
        ldxb = (uint64_t)a.ldx * ES;
        if constexpr (MASK) {
            const size_t block = (size_t)a.n_cols * sizeof(uint2);
            bits = reinterpret_cast<const char*>(a.x_mask) + (size_t)(c0 / 64) * block;
            next_bits = c0 + 64 < a.d ? block : 0;
            bit = lig;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int col = (v * LANES + lig) * VEC;
            ok[v] = col < w;
            const int at = ok[v] ? min(col, w - VEC) : 0;       // (may reach left of c0, never left of column 0: d >= VEC)
            shift[v] = ok[v] ? col - at : 0;
            ok[v] = ok[v] && lig_ < LANES;                      // only the first half stores
            lane_off[v] = (uint32_t)(max(c0 + at, 0) * ES);
        }
    }
    // what a lane keeps of a non-zero: byte offset of its X row (the column itself in the WIDE and MASK forms)
    __device__ __forceinline__ uint32_t key(int32_t c) const { return WIDE || MASK ? (uint32_t)c : (uint32_t)c * (uint32_t)ldxb; }

    // step T's entry: slot T of the group, or slots 2T and 2T+1 for its two halves
    template <int T> static __device__ __forceinline__ uint32_t slot(uint32_t x)
    {
        if constexpr (LANES == 16) return row_bcast<T>(x);
        constexpr int LO = GROUP == 16 ? 2 * T : T, HI = GROUP == 16 ? 2 * T + 1 : 8 + T;      // DPP lanes for its halves
        return (uint32_t)__builtin_amdgcn_update_dpp((int)row_bcast<LO>(x), (int)x, 0x150 + HI, 0xf, 0xc, false);
    }
    template <int T> __device__ __forceinline__ void load(uint32_t key_, Raw<RAW> (&x)[NV]) const
    {
        const uint32_t b = slot<T>(key_);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if constexpr (WIDE) raw_load<BYTES>(X + ((uint64_t)b * ldxb + lane_off[v]), x[v]);
            else raw_load<BYTES>(X + (size_t)(b + lane_off[v]), x[v]);
        }
    }
    template <int T> __device__ __forceinline__ void add(float val, const Raw<RAW> (&x)[NV], float (&acc)[N], const uint2 (&m)[NV]) const
    {
        const float w = __uint_as_float(slot<T>(__float_as_uint(val)));
        if constexpr (MASK) {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const uint32_t lo = row_bcast<T>(m[v].x), hi = row_bcast<T>(m[v].y);
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    const uint32_t on = (uint32_t)__builtin_amdgcn_sbfe((int)(i < 2 ? lo : hi), bit + (i & 1) * 16, 1);     // all ones or zero
                    acc[v * VEC + i] = fmaf(w, __uint_as_float(x[v].w[i] & on), acc[v * VEC + i]);
                }
            }
            return;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[v * VEC + i] = fmaf(w, widened<XK>(x[v].w, i), acc[v * VEC + i]);
    }
    // Steps T0 .. T0+COUNT-1: the rows requested together, then multiplied.  With FIXED the order is fixed here: left alone the compiler
    // widens the first 16-bit row, and waits for it, before it asks for the others (communities, bf16: 64 columns 26.0 -> 23.0
    // us, 128 columns 48.9 -> 34.5 us; f16, 64 columns: 37.6 -> 24.1 us; power law of 169,343 rows, f16, 64 columns: 41 -> 33 us).
    // 16-bit rows of a word per lane and less that take a wave or more each have little to widen and lose by it (bf16, order
    // fixed / left alone: 4,875 rows of 196, 32 columns 9.05 / 8.35 us, 6,627 of 137, 16 columns 8.27 / 7.90).
    static constexpr bool FIXED_WAVE = XK == 0 || BYTES > 4;
    template <bool FIXED, int T0, int COUNT, class Next> __device__ __forceinline__ void steps(uint32_t key_, float val, float (&acc)[N], const uint2 (&m)[NV], Next&& next) const
    {
        Raw<RAW> x[COUNT][NV];
        unrolled<COUNT>([&](auto u) { this->template load<T0 + decltype(u)::value>(key_, x[decltype(u)::value]); });
        if constexpr (FIXED) __builtin_amdgcn_sched_barrier(0);
        if constexpr (T0 == 0) {
            next();
            if constexpr (FIXED) __builtin_amdgcn_sched_barrier(0);
        }
        unrolled<COUNT>([&](auto u) { this->template add<T0 + decltype(u)::value>(val, x[decltype(u)::value], acc, m); });
    }
    // Up to GROUP non-zeros (cnt of them, uniform within the group), U steps at a time.  Slots past the row's end carry the
    // row's last column with value 0, so the loads carry no branches.
    // next(): requests the next batch's indices, behind the first X rows: loads come back in order, and indices, which
    // mostly come from behind L2, would hold up X rows that hit it.
    template <bool FIXED = true, class Next> __device__ __forceinline__ void batch(uint32_t key_, float val, int cnt, float (&acc)[N], Next&& next) const
    {
        uint2 m[NV] = {};
        if constexpr (MASK) {
#pragma unroll
            for (int v = 0; v < NV; ++v) m[v] = *reinterpret_cast<const uint2*>(bits + v * next_bits + (size_t)(key_ * (uint32_t)sizeof(uint2)));
            key_ *= (uint32_t)ldxb;
            if constexpr (FIXED) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (SPLIT == 2 && XK == 0) {
            // a wave whose groups all have more than half a batch left keeps the whole batch in flight (16-bit rows have twice
            // the accumulators and would spill)
            if (__all(cnt > GROUP / 2)) { steps<FIXED, 0, STEPS>(key_, val, acc, m, next); return; }
        }
        unrolled<STEPS / U>([&](auto blk) {
            constexpr int T0 = decltype(blk)::value * U;
            if (T0 == 0 || cnt > T0 * SPLIT) this->template steps<FIXED, T0, U>(key_, val, acc, m, next);
        });
    }
    // (key, value) of non-zero k of a row ending at e (k may run past the end: value 0, last column)
    __device__ __forceinline__ void fetch(const SpmmArgs& a, int k, int e, uint32_t& key_, float& v) const
    {
        const int kc = min(k, e - 1);
        int32_t c;
        float t;
        if constexpr (WIDE || PANEL || (XK == 0 && VEC == 1 && LANES == 16)) {      // (the last ones: 31,552 rows of 45, 16 columns 6.79 us, 6.84 with 32-bit offsets)
            c = a.colind[kc];
            t = a.vals[kc];
        } else {                                                // (32-bit byte offsets: up to 2^30 non-zeros, see launch_csr)
            const size_t at = (uint32_t)kc * 4u;
            c = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(a.colind) + at);
            t = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.vals) + at);
        }
        key_ = key(c);
        v = k < e ? t : 0.f;
    }
    // a span [kb, ke) of one row taken GROUP non-zeros at a time with stride `stride` (GROUP when one group owns the span);
    // EARLY: the next batch's indices are requested before the first X rows
    template <bool FIXED = true, bool EARLY = false> __device__ __forceinline__ void span(const SpmmArgs& a, int kb, int ke, int stride, int lig, float (&acc)[N]) const
    {
        if (kb >= ke) return;
        uint32_t mk, nk;
        float mv, nv;
        fetch(a, kb + lig, ke, mk, mv);
        for (int k0 = kb; k0 < ke; k0 += stride) {
            if constexpr (EARLY) fetch(a, k0 + stride + lig, ke, nk, nv);
            this->template batch<FIXED>(mk, mv, min(GROUP, ke - k0), acc, [&] { if constexpr (!EARLY) fetch(a, k0 + stride + lig, ke, nk, nv); });
            mk = nk;
            mv = nv;
        }
    }
    // a row is done: the two halves' sums are added (the first half's lanes hold the result)
    static __device__ __forceinline__ void finish(float (&acc)[N])
    {
        if constexpr (SPLIT == 2) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                acc[i] += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(acc[i]), 0x128 /* row_ror:8 */, 0xf, 0xf, true));
                if constexpr (!PANEL) asm volatile("" : "+v"(acc[i]));      // (one instruction here, two behind the branch of the store)
            }
        }
    }
    static __device__ __forceinline__ void extent(const SpmmArgs& a, int32_t row, int32_t& s, int32_t& e)
    {
        s = a.rowptr[row];
        e = PANEL ? a.rowend[row] : a.rowptr[row + 1];
    }
    // a panel's share of a row that adds nothing to rows of sums
    static __device__ __forceinline__ bool skipped(const CsrWork& wk, int32_t s, int32_t e) { return PANEL && wk.skip_empty && s == e; }
    // stores the lane's columns of output row `row` (element type a.y_dtype); c0: first column of the slice
    __device__ __forceinline__ void store(const SpmmArgs& a, int y_vec, int64_t row, int c0, int lig, const float (&acc)[N]) const
    {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (!ok[v]) continue;
            const int64_t off = row * a.ldy + c0 + (v * LANES + lig) * VEC - shift[v];
            float y[VEC];
#pragma unroll
            for (int i = 0; i < VEC; ++i) y[i] = acc[v * VEC + i];
            if (PANEL && a.acc) {                               // (the row has VEC columns at this place: see init)
                const f32_any<VEC> t = *reinterpret_cast<const f32_any<VEC>*>(a.acc + row * a.ldacc + (off - row * a.ldy));
#pragma unroll
                for (int i = 0; i < VEC; ++i) y[i] += t.v[i];
            }
            if (y_vec && shift[v] == 0) {
                out_store<VEC, XK != 0 && NV == 1 && !PANEL>(a.Y, a.y_dtype, off, y, a.relu);
            } else {
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    const float one[1] = {y[i]};
                    if (i >= shift[v]) out_store<1, XK != 0 && NV == 1 && !PANEL>(a.Y, a.y_dtype, off + i, one, a.relu);
                }
            }
        }
    }
    // the same into a row of fp32 partial sums (or an LDS tile) starting at p
    __device__ __forceinline__ void store_f32(float* p, int lig, const float (&acc)[N]) const
    {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (!ok[v]) continue;
            float* q = p + (v * LANES + lig) * VEC - shift[v];
#pragma unroll
            for (int i = 0; i < VEC; ++i)
                if (i >= shift[v]) q[i] = acc[v * VEC + i];
        }
    }
};

// ---- mid rows: one wave per row -------------------------------------------------------------
template <class G>
__device__ __forceinline__ void csr_mid_body(uint32_t block, int c_begin, int c_end, const CsrWork& wk, const SpmmArgs& a,
                                             int min_len = 0 /* rows this short belong to another tier */)
{
    const uint32_t item = block * 4 + (threadIdx.x >> 6);
    if (item >= (uint32_t)wk.n_mid) return;
    const int32_t row = wk.mid_rows ? wk.mid_rows[item] : (int32_t)item;
    int32_t s, e;
    G::extent(a, row, s, e);
    if (wk.mid_rows ? e - s <= min_len : e - s > wk.mid_row || (wk.route && wk.route[row / kH] != 0) || G::skipped(wk, s, e)) return;
    const int lane = threadIdx.x & 63, gi = lane / G::GROUP, lig = lane % G::GROUP;
    for (int c0 = c_begin; c0 < c_end; c0 += G::COLS) {
        G g;
        g.init(a, c0, min(G::COLS, c_end - c0), lig);
        float acc[G::N];
        vzero(acc);
        g.template span<G::FIXED_WAVE>(a, s + gi * G::GROUP, e, 64, lig, acc);
        G::finish(acc);
        // butterfly over the groups: same operation order on every run
#pragma unroll
        for (int off = G::GROUP; off < 64; off <<= 1)
#pragma unroll
            for (int i = 0; i < G::N; ++i) acc[i] += __shfl_xor(acc[i], off, 64);
        if (gi == 0) g.store(a, wk.y_vec, row, c0, lig, acc);
    }
}

// ---- short rows -----------------------------------------------------------------------------
// A group owns a row, or grid.rows_per_group consecutive ones on matrices whose launch would not fit otherwise (the WIDE forms
// serve those: the loop costs the plain ones registers).  Every lane
// reads the row's extent itself (one request per group): handing it round between the loads of the chain, and a row's route
// on plans that have no matrix-path windows, cost 2.5 to 10 % of a launch (communities, bf16, 64 columns: 29.1 -> 26.0 us;
// power law, fp32, 128 columns: 119.5 -> 116.4 us).
template <class G>
__device__ __forceinline__ void csr_short_row(uint32_t i, int lig, int c_begin, int c_end, const CsrWork& wk, const SpmmArgs& a)
{
    const int32_t row = wk.row_list ? wk.row_list[i] : (int32_t)i;
    int32_t s, e;
    G::extent(a, row, s, e);
    // rows owned by the matrix path or by the other tiers
    if (!wk.row_list && ((wk.route && wk.route[row / kH] != 0) || e - s > wk.mid_row)) return;
    if (G::skipped(wk, s, e)) return;
    for (int c0 = c_begin; c0 < c_end; c0 += G::COLS) {
        G g;
        g.init(a, c0, min(G::COLS, c_end - c0), lig);
        float acc[G::N];
        vzero(acc);
        g.span(a, s, e, G::GROUP, lig, acc);
        G::finish(acc);
        g.store(a, wk.y_vec, row, c0, lig, acc);
    }
}
template <class G>
__device__ __forceinline__ void csr_short_body(uint32_t block, int c_begin, int c_end, const CsrWork& wk, const SpmmArgs& a)
{
    const int lig = threadIdx.x % G::GROUP;
    const uint32_t group = block * (256 / G::GROUP) + threadIdx.x / G::GROUP;
    if constexpr (G::MANY) {
        const uint32_t i0 = group * wk.grid.rows_per_group, i1 = min(i0 + (uint32_t)wk.grid.rows_per_group, (uint32_t)wk.n_items);
        for (uint32_t i = i0; i < i1; ++i) csr_short_row<G>(i, lig, c_begin, c_end, wk, a);
    } else if (group < (uint32_t)wk.n_items) {
        csr_short_row<G>(group, lig, c_begin, c_end, wk, a);
    }
}

// ---- short rows with the update stage fused in ------------------------------------------------
// Same walk as csr_short_body, but a workgroup covers exactly one list entry per group (16 or 32) and a finished row goes to
// one of one or two 16 x d tiles in LDS instead of memory; after a barrier the four waves share the tiles, each multiplying
// one by an interleaved quarter or half of W's 16-column blocks on the matrix cores, and write act(Z W) for the rows the workgroup owns
// (Section V-A: the aggregation result of a window stays on chip for the update).
// The width d must fit one pass of the group (d <= G::COLS) and be a multiple of 16.
template <class G>
__device__ __forceinline__ void csr_short_fused_body(uint32_t block, const CsrWork& wk, const SpmmArgs& a, const UpdateArgs& u,
                                                     float* __restrict__ zt, int32_t* __restrict__ rows_s)
{
    constexpr int LDZ = G::COLS + 4, ROWS = 256 / G::GROUP, WPT = 64 / ROWS;   // waves per tile
    const uint32_t b0 = block * ROWS;                           // first list entry of the workgroup
    if (b0 >= (uint32_t)wk.n_items) return;                               // whole workgroup past the end
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int gw = threadIdx.x / G::GROUP, lig = threadIdx.x % G::GROUP;
    int32_t row = -1, k = 0, e = 0;                             // (the fused launch has no list)
    if (b0 + gw < (uint32_t)wk.n_items) {
        row = (int32_t)(b0 + gw);
        G::extent(a, row, k, e);
        if ((wk.route && wk.route[row / kH] != 0) || e - k > wk.mid_row) row = -1;
    }
    if (lig == 0) rows_s[gw] = row;
    G g;
    g.init(a, 0, a.d, lig);
    if (row >= 0) {
        float acc[G::N];
        vzero(acc);
        // (rows of 65 to 128 bytes of fp32, where one group's chain of batches holds up the tile, behind their rows / before: 2,240 rows
        // of 40, 32 -> 64: 16.2 / 14.1 us, 1.2 M of 55, 32 -> 32: 1003 / 991)
        g.template span<true, G::ES == 4 && G::LANES == 8>(a, k, e, G::GROUP, lig, acc);
        G::finish(acc);
        g.store_f32(zt + gw * LDZ, lig, acc);
    }
    __syncthreads();
    if (u.keep_z) store_tile_rows(zt, LDZ, rows_s, ROWS, a.d, a.Y, a.ldy, threadIdx.x, 256);
    const int tile = wave / WPT;
    update_tile16(zt + tile * 16 * LDZ, LDZ, rows_s + tile * 16, a.d, u, lane, wave % WPT, WPT);
}

// ---- long rows: one workgroup per segment of a row ------------------------------------------
template <class G>
__device__ __forceinline__ void csr_long_body(uint32_t block, int c_begin, int c_end, const CsrWork& wk,
                                              float* __restrict__ red /* LDS, 256 * G::N floats */, const SpmmArgs& a)
{
    constexpr int NG = 256 / G::GROUP;
    if (block >= (uint32_t)wk.n_segs) return;
    const Segment sg = wk.segs[block];
    const int gi = threadIdx.x / G::GROUP, lig = threadIdx.x % G::GROUP;
    for (int c0 = c_begin; c0 < c_end; c0 += G::COLS) {
        G g;
        g.init(a, c0, min(G::COLS, c_end - c0), lig);
        float acc[G::N];
        vzero(acc);
        g.template span<G::FIXED_WAVE>(a, sg.k_begin + gi * G::GROUP, sg.k_end, 256, lig, acc);
        G::finish(acc);
        // fixed-order tree over the groups: the result does not depend on scheduling
#pragma unroll
        for (int i = 0; i < G::N; ++i) red[i * 256 + threadIdx.x] = acc[i];
        __syncthreads();
        for (int st = NG / 2; st > 0; st >>= 1) {
            if (gi < st) {
#pragma unroll
                for (int i = 0; i < G::N; ++i) red[i * 256 + threadIdx.x] += red[i * 256 + threadIdx.x + st * G::GROUP];
            }
            __syncthreads();
        }
        if (gi == 0) {
#pragma unroll
            for (int i = 0; i < G::N; ++i) acc[i] = red[i * 256 + lig];
            if (sg.slot < 0) g.store(a, wk.y_vec, sg.row, c0, lig, acc);
            else g.store_f32(wk.partial + (int64_t)sg.slot * a.d + c0, lig, acc);
        }
        __syncthreads();
    }
}

// ---- one launch for all three tiers ---------------------------------------------------------
template <class G>
__device__ __forceinline__ void csr_body(const CsrWork& wk, const SpmmArgs& a, float* __restrict__ red /* LDS, 256 * G::N floats */)
{
    uint32_t b = blockIdx.x;
    int slice;
    if (b < wk.grid.seg_blocks * wk.grid.n_slices) {
        b = csr_block(blockIdx.x, b, wk.grid.seg_blocks, -1, wk.grid.n_slices, slice);
        const int c0 = slice * wk.grid.slice_w;
        csr_long_body<G>(b, c0, min(a.d, c0 + wk.grid.slice_w), wk, red, a);
        return;
    }
    b -= wk.grid.seg_blocks * wk.grid.n_slices;
    if (b < wk.grid.mid_blocks * wk.grid.n_slices) {
        b = csr_block(blockIdx.x, b, wk.grid.mid_blocks, wk.grid.run_mid, wk.grid.n_slices, slice);
        const int c0 = slice * wk.grid.slice_w;
        csr_mid_body<G>(b, c0, min(a.d, c0 + wk.grid.slice_w), wk, a);
        return;
    }
    b -= wk.grid.mid_blocks * wk.grid.n_slices;
    b = csr_block(blockIdx.x, b, wk.grid.short_blocks, wk.grid.run, wk.grid.n_slices, slice);
    const int c0 = slice * wk.grid.slice_w;
    csr_short_body<G>(b, c0, min(a.d, c0 + wk.grid.slice_w), wk, a);
}
template <class G>
__global__ __launch_bounds__(256, G::WAVES) void k_csr(CsrWork wk, SpmmArgs a)
{
    __shared__ float red[256 * G::N];
    csr_body<G>(wk, a, red);
}
// The same with MOST waves per SIMD and no more, which the register allocation is rounded up for (few_waves says when; LDS to the
// same end is held until a workgroup's last wave is done: 2,383 us where this takes 2,225).
template <class G, int MOST>
__global__ __attribute__((amdgpu_flat_work_group_size(1, 256), amdgpu_waves_per_eu(1, MOST))) void k_csr_few(CsrWork wk, SpmmArgs a)
{
    __shared__ float red[256 * G::N];
    csr_body<G>(wk, a, red);
}

// The launch of a matrix of few rows, all of them mid or long rows (see launch_csr): what a call passes is held to 112 bytes.  Beyond that a
// launch costs the host 0.9 us more (2.7 us up to 112 bytes of arguments, 3.6 from 120 on, kernels of nothing), and these calls are little else: 2,708 rows of 5, 32
// columns, calls in a row 4.0 -> 3.5 us (4.8 -> 4.6 through the Python binding).
struct CsrFewRows {
    const int32_t *rowptr, *colind;
    const float* vals;
    const void* X;
    float* Y;
    const Segment* segs;
    float* partial;
    int32_t ldx, ldy, n_rows, d, long_row, n_segs;
    uint32_t seg_blocks, mid_blocks;
    int32_t run_mid, slice_w;
    uint8_t n_slices, y_dtype, relu, y_vec;
};
static_assert(sizeof(CsrFewRows) <= 112, "arguments of a cheap launch");
template <class G>
__global__ __launch_bounds__(256, G::WAVES) void k_csr_few_rows(CsrFewRows r)
{
    __shared__ float red[256 * G::N];
    SpmmArgs a{};
    a.n_rows = r.n_rows; a.rowptr = r.rowptr; a.colind = r.colind; a.vals = r.vals; a.X = r.X; a.ldx = r.ldx; a.d = r.d;
    a.Y = r.Y; a.ldy = r.ldy; a.relu = r.relu; a.y_dtype = r.y_dtype;
    CsrWork wk{};
    wk.n_segs = r.n_segs; wk.segs = r.segs; wk.partial = r.partial; wk.n_mid = r.n_rows; wk.mid_row = r.long_row; wk.y_vec = r.y_vec;
    uint32_t b = blockIdx.x;
    int slice;
    if (b < r.seg_blocks * r.n_slices) {
        b = csr_block(blockIdx.x, b, r.seg_blocks, -1, r.n_slices, slice);
        const int c0 = slice * r.slice_w;
        csr_long_body<G>(b, c0, min(a.d, c0 + r.slice_w), wk, red, a);
        return;
    }
    b -= r.seg_blocks * r.n_slices;
    b = csr_block(blockIdx.x, b, r.mid_blocks, r.run_mid, r.n_slices, slice);
    const int c0 = slice * r.slice_w;
    csr_mid_body<G>(b, c0, min(a.d, c0 + r.slice_w), wk, a);
}

// The same launch with the update stage fused into the short rows; long and mid rows write their
// aggregated rows to a.Y (the workspace Z) and are finished by k_update_rest.
// (Four waves per SIMD for 16-bit rows of 129 to 256 bytes, whose form the compiler else gives a few registers too many: 1.2 M rows of
// 55, bf16, 128 -> 128: 2,438 -> 2,372 us.)
template <class G>
__global__ __launch_bounds__(256, G::ES == 2 && G::BYTES == 16 && G::N == 8 && G::LANES == 16 ? 4 : 1) void k_csr_fused(CsrWork wk, SpmmArgs a, UpdateArgs u)
{
    constexpr int kTile = 256 / G::GROUP * (G::COLS + 4), kRed = 256 * G::N;
    __shared__ float lds[kTile > kRed ? kTile : kRed];          // the reduction of a long row and the tile of short rows never meet
    __shared__ int32_t rows_s[256 / G::GROUP];
    uint32_t b = blockIdx.x;
    int slice;
    if (b < wk.grid.seg_blocks) {
        csr_long_body<G>(b, 0, a.d, wk, lds, a);
        return;
    }
    b -= wk.grid.seg_blocks;
    if (b < wk.grid.mid_blocks) {
        csr_mid_body<G>(b, 0, a.d, wk, a, wk.mid_row);          // the fused tier takes rows up to mid_row
        return;
    }
    b -= wk.grid.mid_blocks;
    b = csr_block(blockIdx.x, b, wk.grid.short_blocks, wk.grid.run, 1, slice);
    csr_short_fused_body<G>(b, wk, a, u, lds, rows_s);
}

// ---- rows the fused kernels did not finish: gather their aggregated rows and apply the update ---
// One wave per 16 entries of the plan's list of such rows (rows of matrix-path windows wider than
// the wave-per-window kernel handles, scalar-path rows above the short tier): they were written to
// Z, are read back as a 16-row tile and multiplied by W.
// NT: output columns per lane and pass (chosen on the host by update_tile_nt; a narrower NT needs fewer registers,
// which is what bounds the waves in flight of this streaming kernel).
template <int ZD, int NT>
__global__ __launch_bounds__(256) void k_update_rest(int32_t n_rest, const int32_t* __restrict__ rest_rows, int tiles_per_wave,
                                                     SpmmArgs a, UpdateArgs u)
{
    constexpr int ldz = ZD + 4;                                 // ZD >= d
    __shared__ float tiles[4 * 16 * ldz];
    __shared__ int32_t rows_s[2][64];                           // two row lists per wave, alternating between tiles
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t n_tiles = ((int64_t)n_rest + 15) / 16;
    const int64_t t_begin = ((int64_t)blockIdx.x * 4 + wave) * tiles_per_wave;
    const int64_t t_end = min(n_tiles, t_begin + tiles_per_wave);
    if (t_begin >= t_end) return;
    float* __restrict__ zt = tiles + wave * 16 * ldz;
    constexpr int kPerLane = 16 * ZD / 4 / 64;                  // float4 per lane for the widest tile
    const int per_row = a.d >> 2;
    float4 v[kPerLane];
    // A wave walks tiles_per_wave consecutive 16-row tiles.  The whole 16 x d tile is requested at once, all lanes busy;
    // the next tile's rows are requested as soon as the current tile is parked in LDS, so they arrive during its MFMAs.
    auto request = [&](int64_t tile, int32_t* __restrict__ rows16) {
        const int64_t i0 = tile * 16;
        if (lane < 16) rows16[lane] = i0 + lane < n_rest ? rest_rows[i0 + lane] : -1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const int idx = lane + 64 * j;
            v[j] = make_float4(0.f, 0.f, 0.f, 0.f);             // tile rows past the list are zero and never stored
            if (idx < 16 * per_row) {
                const int32_t rr = rows16[idx / per_row];
                if (rr >= 0) v[j] = *reinterpret_cast<const float4*>(&a.Y[(int64_t)rr * a.ldy + (idx % per_row) * 4]);
            }
        }
    };
    request(t_begin, rows_s[0] + wave * 16);
    for (int64_t t = t_begin; t < t_end; ++t) {
        int32_t* __restrict__ rows16 = rows_s[(t - t_begin) & 1] + wave * 16;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const int idx = lane + 64 * j;
            if (idx < 16 * per_row) *reinterpret_cast<float4*>(&zt[(idx / per_row) * ldz + (idx % per_row) * 4]) = v[j];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (t + 1 < t_end) request(t + 1, rows_s[(t + 1 - t_begin) & 1] + wave * 16);
        update_tile16_nt<NT>(zt, ldz, rows16, a.d, u, lane, 0, 1);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the tile's LDS reads are done before it is overwritten
    }
}

// ---- rows cut into several segments: add the partial rows in segment order ------------------
// A launch of little else than three trips to memory: the record, the partial rows, eight of them requested together whatever their
// number (one after the other a row of seven segments makes nine trips), the sums of earlier panels beside them.  (Whole calls are level.)
__global__ __launch_bounds__(256) void k_reduce_partials(int32_t n_multi, const MultiRow* __restrict__ multi,
                                                         const float* __restrict__ partial, SpmmArgs a)
{
    const MultiRow m = multi[blockIdx.x];
    for (int c = threadIdx.x; c < a.d; c += 256) {
        float acc = 0.f;
        const float before = a.acc ? a.acc[(int64_t)m.row * a.ldacc + c] : 0.f;
        for (int q0 = 0; q0 < m.n_slots; q0 += 8) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = partial[(int64_t)(m.first_slot + min(q0 + q, m.n_slots - 1)) * a.d + c];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc += q0 + q < m.n_slots ? v[q] : 0.f;
        }
        if (a.acc) acc += before;
        const float one[1] = {acc};
        out_store<1>(a.Y, a.y_dtype, (int64_t)m.row * a.ldy + c, one, a.relu);
    }
}

// ---- dispatch ---------------------------------------------------------------------------------
struct CsrShape { int vec, nv, lanes, group; bool wide; };

// Vectors of up to 16 bytes per lane: 8 lanes per row for rows of 65 to 128 bytes (two rows at a time, see Gather), 16 lanes
// otherwise, with 4 bytes (2 for 16-bit X) each for the narrow rows and several vectors each for the wide ones.  A row of X
// needs no more than 4-byte alignment for that; 16-bit X with odd rows or an odd base is read element by element.
// narrow: rows of up to 128 bytes in the form of 8 lanes to an output row, if their alignment allows it.
static CsrShape pick_shape(const SpmmArgs& a, bool narrow)
{
    const bool f32 = a.x_dtype == HCSPMM_F32;
    const int es = f32 ? 4 : 2, per16 = 16 / es;
    CsrShape sh{1, 1, 16, 16, false};
    if (f32 || (a.d % 2 == 0 && a.ldx % 2 == 0 && (uintptr_t)a.X % 4 == 0)) {
        if (narrow && a.d * es <= 128) {
            sh.lanes = sh.group = 8;
            sh.vec = 4 / es;
            while (8 * sh.vec < a.d) sh.vec *= 2;
        } else if (a.d * es > 64) {
            sh.vec = per16;
            if (a.d * es <= 128) sh.lanes = 8;
        } else {
            while (sh.vec < per16 && 16 * sh.vec < a.d) sh.vec *= 2;
        }
    }
    const int most = f32 ? 4 : (sh.vec == 1 ? 4 : 2);
    while (sh.nv < most && sh.lanes * sh.vec * sh.nv < a.d) sh.nv *= 2;
    if (!f32 && sh.vec == 1 && sh.nv > 1) sh.nv = 4;
    // 32-bit byte offsets reach 4 GiB of X (the last row is read to its end)
    sh.wide = ((uint64_t)(a.n_cols > 0 ? a.n_cols - 1 : 0) * (uint64_t)a.ldx + (uint64_t)a.d) * es >= ((uint64_t)1 << 32);
    return sh;
}
static int shape_cols(const CsrShape& sh) { return sh.lanes * sh.vec * sh.nv; }

// FN(element kind, vector, vectors, lanes, group, wide)
#define HC_CSR_ONE(FN, XK, V, NVV, L, GR) do { if (sh.wide) { FN(XK, V, NVV, L, GR, true); } else { FN(XK, V, NVV, L, GR, false); } } while (0)
#define HC_CSR_PANEL_DISPATCH(FN, XK, V)                                                           \
    if (sh.lanes == 8) HC_CSR_ONE(FN, XK, V, 1, 8, 16);                                            \
    else if (sh.nv == 1) HC_CSR_ONE(FN, XK, V, 1, 16, 16);                                         \
    else HC_CSR_ONE(FN, XK, V, 2, 16, 16);
#define HC_CSR_DISPATCH32_16(FN)                                                                   \
    if (sh.vec == 1) HC_CSR_ONE(FN, 0, 1, 1, 16, 16);                                              \
    else if (sh.lanes == 8) HC_CSR_ONE(FN, 0, 4, 1, 8, 16);                                        \
    else if (sh.nv == 1) HC_CSR_ONE(FN, 0, 4, 1, 16, 16);                                          \
    else if (sh.nv == 2) HC_CSR_ONE(FN, 0, 4, 2, 16, 16);                                          \
    else HC_CSR_ONE(FN, 0, 4, 4, 16, 16);
#define HC_CSR_DISPATCH32(FN)                                                                      \
    if (sh.group == 8) {                                                                           \
        if (sh.vec == 1) HC_CSR_ONE(FN, 0, 1, 1, 8, 8);                                            \
        else if (sh.vec == 2) HC_CSR_ONE(FN, 0, 2, 1, 8, 8);                                       \
        else HC_CSR_ONE(FN, 0, 4, 1, 8, 8);                                                        \
    } else { HC_CSR_DISPATCH32_16(FN) }
#define HC_CSR_DISPATCH16(FN, XK)                                                                  \
    if (sh.group == 8) {                                                                           \
        if (sh.vec == 2) HC_CSR_ONE(FN, XK, 2, 1, 8, 8);                                           \
        else if (sh.vec == 4) HC_CSR_ONE(FN, XK, 4, 1, 8, 8);                                      \
        else HC_CSR_ONE(FN, XK, 8, 1, 8, 8);                                                       \
    } else if (sh.vec == 1) { if (sh.nv == 1) HC_CSR_ONE(FN, XK, 1, 1, 16, 16); else HC_CSR_ONE(FN, XK, 1, 4, 16, 16); }  \
    else if (sh.vec == 2) HC_CSR_ONE(FN, XK, 2, 1, 16, 16);                                        \
    else if (sh.lanes == 8) HC_CSR_ONE(FN, XK, 8, 1, 8, 16);                                       \
    else if (sh.nv == 1) HC_CSR_ONE(FN, XK, 8, 1, 16, 16);                                         \
    else HC_CSR_ONE(FN, XK, 8, 2, 16, 16);
#define HC_CSR_DISPATCH(FN)                                                                        \
    if (a.x_dtype == HCSPMM_F32) { HC_CSR_DISPATCH32(FN) }                                         \
    else if (a.x_dtype == HCSPMM_BF16) { HC_CSR_DISPATCH16(FN, 1) }                                \
    else { HC_CSR_DISPATCH16(FN, 2) }

// Column slices.  More than 512 bytes of a row per lane group would cost the registers that keep enough loads in flight
// (fp32, 256 columns, 30,000 nodes: 138 us in one slice of four vectors per lane, 57 us in two slices), so wider rows are
// always cut.  Beyond that, slices trade index and row-offset traffic (8 bytes per non-zero and slice) and one more set of
// row chains for L2 hits: an XCD that works on one slice of every row keeps twice or four times as many rows of it.  That
// pays where an X row is read often compared with the size of X -- measured on power-law graphs, fp32, 128 columns:
// 30,000 nodes of degree 20: 37.7 -> 25.1 us with two slices, 169,000 of 15: 118 -> 111 us, 500,000 of 60: 1973 -> 1850 us
// and 1754 us with four; but 500,000 of degree 6: 261 -> 285 us, 2.4 M of 51: 8.63 -> 8.69 ms -- i.e. from about five
// non-zeros per row for every 64 MiB of X.  128-byte slices win over 256-byte ones from about 40 non-zeros per row (the
// per-row chain is then small; 60,000 nodes of degree 100: 271 / 228 / 201 us with 1 / 2 / 4 slices), as long as rows of X
// start on a 128-byte line: off it, every slice costs a second line (300,000 of degree 60, bf16, 224 columns: 1345 us in
// four slices, 256 columns 969 us).  Neighbouring rows that share their columns (community graphs) already meet in one L2
// and lose 6 to 27 %: they are left whole.
// 16-bit rows of more than 256 and less than 512 bytes leave lanes of the two-vector form idle, at half the waves: three
// slices of 128 bytes where rows start on lines (16,934 nodes of 14, 192 columns, bf16: 26 -> 17 us; 1 M of 20: 1207 -> 1094 us),
// two halves while X fits the L2s (16,934 of 14, 160 columns: 25 -> 15 us; 100,000 of 20: 91 -> 92 us).  Whole 16-bit rows of
// 512 bytes are slow where most rows take a wave each, also where nothing is gained in L2 (communities of 512, 232,960 rows
// of 165, bf16: 1268 -> 922 us in halves).
// fp32 rows of more than 512 and up to 1024 bytes off the 128-byte lines: a cut costs every row another line, and where the X
// rows come from behind L2 the whole row in four vectors per lane wins although fewer loads are in flight -- earlier where two
// halves of whole lines are uneven or rows are not even on half lines (two slices / whole, us, 200 columns: 100,000 rows of 60:
// 652 / 552, 478,000 of 93: 6454 / 4795, 1 M of 20: 2810 / 2402; 130 columns: 100,000 of 20: 182 / 148; but 50,000 of 60: 260 /
// 266) than where they are (240 columns: 70,000 of 60: 398 / 425, 300,000 of 60: 2381 / 2100, 1 M of 6: 1117 / 1136).
// Communities share their rows in L2 and take whole rows on the largest X only (300,000 of 29, 200 columns: 544 / 478 us;
// 131,072 of 51: 248 / 257), and up to 768 bytes slices of 256 bytes, which need one vector per lane (131,072 of 51, 144
// columns: 220 -> 182 us, 160 columns: 215 -> 175 us).
static int pick_slices(const SpmmArgs& a, const CsrHints& h, int32_t& slice_w)
{
    const int64_t es = a.x_dtype == HCSPMM_F32 ? 4 : 2, row = a.d * es;
    const bool on_lines = a.ldx * es % 128 == 0 && (uintptr_t)a.X % 128 == 0;
    int64_t most = 512, align = 128 / es;                       // bytes of a row per slice; slices of whole 128-byte lines
    const double degree = h.rows > 0 ? (double)h.nnz / (double)h.rows : 0.0;
    const bool often = h.scattered && degree >= 5.0 * ((double)a.n_cols * (double)row / (64.0 * (1 << 20)));
    if (often && on_lines && degree >= 40.0 && row >= 256) most = 128;
    else if (often && row >= 512) most = 256;
    else if (es == 2 && h.scattered && row > 256 && row < 512) {
        if (on_lines) most = 128;
        else if ((double)a.n_cols * (double)row <= 20.0 * (1 << 20)) { most = 256; align = 32; }
    } else if (es == 2 && row >= 512 && degree > kMidRow) {
        most = 256;
    }
    if (es == 4 && row > 512 && row <= 1024) {
        const double x_mb = (double)a.n_cols * (double)row / (1 << 20);
        const bool uneven = a.ldx * es % 64 != 0 || 10 * ((a.d + 63) / 64 * 32) > 6 * a.d;
        const bool whole = h.scattered ? x_mb >= 48.0 && (uneven || (x_mb >= 96.0 && degree >= 15.0)) : x_mb >= 200.0 && row > 768;
        if (!on_lines && whole) most = 1024;
        else if (!h.scattered && row <= 768) most = 256;
    }
    int64_t n = (row + most - 1) / most;
    // a count that XCDs can own, where the slices come out about equally wide; other counts are taken in turn (as are the
    // narrow slices of rows that share what they read: nothing is gained by owners)
    for (int64_t m = n; m > 1 && n < 8 && (row + m - 1) / m <= 512 && !(most == 256 && !h.scattered); --m) {
        const int64_t w = ((a.d + m - 1) / m + align - 1) / align * align;
        if ((m & (m - 1)) == 0 && 5 * m * w <= 6 * a.d) { n = m; break; }
    }
    slice_w = (int32_t)(((a.d + n - 1) / n + align - 1) / align * align);
    const int n_slices = (int)((a.d + slice_w - 1) / slice_w);
    if (n_slices <= 1) slice_w = a.d;
    return n_slices;
}

// With the update fused in, a workgroup of 8-lane groups has 32 rows to multiply instead of 16, at the same barrier, loads of W
// and epilogue: 2.4 M rows of 51, 32 -> 32: 2371 -> 2165 us, 300,000 of 20: 141 -> 111 us.  A graph that is all launches
// prefers the shorter chains of 16 (2,708 rows: 6.9 us against 8.6 us).
static bool fused_narrow(const SpmmArgs& a) { return a.n_rows > kMidRowFewRows; }

// The fused update needs the whole aggregated row in one pass of a lane group and a width that the update's K loop takes
// 16 at a time, and a launch holds 16 rows per workgroup of no more than 2^26 rows (and what mid and long rows they may be).
bool update_fusable(const SpmmArgs& a)
{
    if (a.d % 16 != 0 || a.d < 16 || a.d > 256 || a.n_rows > (1 << 26)) return false;
    const CsrShape sh = pick_shape(a, fused_narrow(a));
    return shape_cols(sh) >= a.d && a.ldy % 4 == 0 && (uintptr_t)a.Y % 16 == 0 && mfma_update_fusable(a);
}

bool csr_panels_usable(const SpmmArgs& a)
{
    const CsrShape sh = pick_shape(a, false);
    return (int64_t)a.d * (a.x_dtype == HCSPMM_F32 ? 4 : 2) >= kPanelRowBytes && sh.vec == (a.x_dtype == HCSPMM_F32 ? 4 : 8);
}

// Where 8 lanes per output row (Gather's third form) are ahead of 16: on matrices of many short rows, which are bound by how
// fast waves start and drain, and where rows of X off the 16-byte pieces make 16 narrow lanes touch more lines than 8 wider
// ones.  On fewer rows the chain of a row that is just short of the wave-per-row tier, twice as long then, outlasts the rest.
// 16 against 8 lanes, us, fp32 (two columns of 16 bits like one of fp32; * off the 16-byte pieces):
//                               8 columns      16 columns     32 columns     7 columns *    9 columns *
//   2.4 M rows of 9             349 / 280      389 / 342      463 / 407      406 / 315      --
//   400,000 of 11               --             60 / 57        92 / 93        --             65 / 54
//   200,000 of 15               --             34 / 33        54 / 56        --             38 / 32
//   169,343 of 15               26.2 / 22.1    28.1 / 28.2    33.1 / 32.5    35.4 / 27.2    --
//   131,072 in communities, 20  17.5 / 13.7    18.6 / 20.7    22.7 / 22.3    28.0 / 19.4    28.1 / 21.0
//   102,271 of 9                --             14.1 / 15.8    19.2 / 21.2    --             17.3 / 15.6
//   1 M of 21                   222 / 213      268 / 263      315 / 319      256 / 233      --
//   50,021 of 29                10.0 / 9.7     12.1 / 14.2    14.6 / 15.8    16.3 / 12.9    --
//   16,934 of 15                4.8 / 5.0      4.8 / 6.1      5.4 / 6.3      6.5 / 5.5      --
//   300,000 of 61               129 / 137      170 / 178      --             161 / 150      --
//   2.4 M of 51                 1607 / 1679    1878 / 1907    2100 / --      1797 / 1835    --
static bool narrow_rows(const SpmmArgs& a, const CsrHints& h)
{
    const int64_t es = a.x_dtype == HCSPMM_F32 ? 4 : 2, row = a.d * es;
    if (row > 128 || h.rows <= 0) return false;
    const double degree = (double)h.nnz / (double)h.rows;
    const bool off = a.ldx * es % 16 != 0 || (uintptr_t)a.X % 16 != 0;
    if (off && row <= 64 && degree < 40.0 && ((es == 4 && row <= 40) || h.rows <= kMidRowFewRows || h.rows >= 130000)) return true;
    if (row <= 32) return h.rows >= 100000 && degree <= 24.0;
    return degree <= 16.0 && h.rows >= (row <= 64 ? 200000 : 1000000);
}

// Waves per SIMD that whole rows of more than 512 bytes of fp32, 256 of 16 bits, are held to on scattered matrices, and others below (0: what the
// registers allow, five to six).  The forms that read them ask for eight vectors per lane at once, and all those waves for more than the
// L2s keep for each other.  Where rows have many non-zeros, which is where X rows are read again, fewer waves are ahead, and
// where they have very many and are wide, two (all / three / two, us, power laws; fp32: 1 M rows of 20, 150 columns: 2428 / 2225 /
// 2361, of 15: 1941 / 1748 / 1903, 300,000 of 60, 200: 2042 / 2014 / 1819, 478,000 of 93, 200: 4900 / 4839 / 4520, 90,000 of 45, 150:
// 282 / 278 / 285; but 800,000 of 13, 172: 1124 / 1141, 400,000 of 6, 140: 261 / 283; bf16: 500,000 of 30, 252: 1152 / 1139, 300,000
// of 60, 200: 1038 / 1029 / 970, f16 200,000 of 45, 160: 345 / 341 / 367; but 2 M of 16, 144: 1780 / 1865, 600,000 of 20, 180: level).
// Beside the matrix path's kernels they are held to three whatever the matrix, which leaves those the room to run at all (all / three,
// us, fp32: 1 M rows of 20, 150 columns: 2433 / 2231, communities + power law, 1.2 M rows, 186: 2030 / 1883, 250: 2554 / 2334), 16-bit
// rows only where those left to this path have 12 non-zeros and more (bf16, 1 M of 20, 136: 1087 / 1058, 184: 1339 / 1311; communities
// + power law, 1.2 M of 20, 200: level, but 2 M of 9, 160: 1304 / 1400, 2.4 M of 7, 144: 1274 / 1443).
// In column panels, whose X rows are meant to stay in the L2s, 16-bit rows are held to three from 168 columns on and to two from 224
// (all / three / two, us, bf16: 104,000 rows of 193, 136 columns: 533 / 559 / 675, 184: 713 / 690 / 753, 252: 1040 / 998 / 985; 66,576
// of 180, 184: 415 / 395 / 409, 252: 603 / 577 / 551; f16 the same).
// Scattered rows of one 16-byte vector per lane, whole or in slices: what all eight waves ask for at once is more than an XCD's L2, and from
// 40 non-zeros per row and 36 MB of X on, where rows come back often enough, five waves find more of it there, from 60 on four, rows of up to 64 columns of 16 bits from 85 on
// (all / five / four, us, fp32: 2.4 M rows of 51, 32 columns: 2116 / 2096 / 2089 (five: 1.1 % fewer bytes behind L2, hits 19.7 -> 20.0 %), 1 M of 43, 32: 649 / 639 / 635, of 51, 64: 1528 / 1525 / 1536, 300,000 of 43, 128: 698 / 688 /
// 693, of 111, 64: 867 / 850 / 840, 400,000 of 76, 64: 838 / 817 / 807, 128: 1744 / 1710 / 1695; but 300,000 of 36, 32: 138 / 139 / 142, 1 M of 21, 32:
// 312 / 326 / 347, 100,000 of 51, 64: 95 / 98 / 104; bf16: 1 M of 51, 64 columns: 816 / 795 / 786, 300,000 of 51, 64: 200 / 195 / 200, 400,000 of 61, 64: 306 / 300 / 308, of 76: 386 / 376 / 379, 700,000 of 90, 64: 873 / 846 /
// 844, 300,000 of 111, 128: 895 / 862 / 841,
// 700,000 of 101, 64: 1058 / 1024 / 1003; but 1 M of 21, 64: 363 / 369 / 388).  Whole rows of up to 128 bytes of fp32 from 96 MB or
// 70 non-zeros on (600,000 of 65, 24 columns: 610 / -- / 615, 300,000 of 42, 32: 163.0 / 163.7 / --), fp32 rows of more than 64 from 60 non-zeros on only (beside
// communities of half the rows, 431,072 of 42, 128: 799 / 809 / --, 300,000 of 42, 128, another graph than above: 634 / 637 / --).
static int few_waves(const SpmmArgs& a, const CsrHints& h, const CsrShape& sh, int32_t width)
{
    const bool f32 = a.x_dtype == HCSPMM_F32;
    if (sh.vec == (f32 ? 4 : 8) && sh.nv == 1 && sh.group == 16 && !sh.wide && !a.rowend && !h.beside && h.scattered) {
        const double x_mb = (double)a.n_cols * a.d * (f32 ? 4 : 2) / (1 << 20);
        if (h.nnz < 40 * h.rows || x_mb < 36.0 || (f32 && a.d <= 32 && x_mb < 96.0 && h.nnz < 70 * h.rows)) return 0;
        if (f32 && a.d > 64 && h.nnz < 60 * h.rows) return 0;
        return h.nnz < (f32 || sh.lanes == 16 ? 60 : 85) * h.rows ? 5 : 4;
    }
    if (sh.lanes != 16 || sh.vec * sh.nv != 16 || !(f32 || sh.vec == 8) || h.rows <= 0) return 0;
    if (a.rowend) return f32 || width < 168 ? 0 : width < 224 ? 3 : 2;
    const double degree = (double)h.nnz / (double)h.rows;
    if (h.beside) return f32 || degree >= 12.0 ? 3 : 0;
    if (!h.scattered) return 0;
    return degree >= 40.0 && a.d >= 168 ? 2 : degree >= (f32 ? 15.0 : 28.0) ? 3 : 0;
}

static bool few_rows_form(const SpmmArgs& a, int n_slices) { return (int64_t)a.n_rows * n_slices <= (a.x_dtype == HCSPMM_F32 ? 4096 : 6144); }

bool csr_mask_usable(const SpmmArgs& a, const CsrHints& hints)
{
    if (a.x_dtype != HCSPMM_F32 || a.d % 4 != 0 || a.d <= 32 || a.rowend || a.acc || hints.beside || hints.entries > ((int64_t)1 << 30) || tune().rpg >= 1) return false;
    if ((int64_t)a.n_cols * (int64_t)sizeof(uint2) > INT32_MAX) return false;
    SpmmArgs t = a;
    int32_t slice_w;
    const int n_slices = pick_slices(a, hints, slice_w);
    if (n_slices > 1) t.d = slice_w;
    const CsrShape sh = pick_shape(t, false);
    if (pick_shape(a, false).wide || sh.vec != 4 || sh.lanes != 16 || sh.nv > 2 || (n_slices > 1 && slice_w % 64 != 0)) return false;
    return !few_rows_form(a, n_slices) && (int64_t)a.n_rows * n_slices <= ((int64_t)1 << 26) && few_waves(a, hints, sh, t.d) == 0;
}

hipError_t launch_csr(const SpmmArgs& a, int32_t n_segs, const Segment* segs, float* partial, int32_t n_mid,
                      const int32_t* mid_rows, int32_t n_items, const int32_t* row_list, const uint8_t* route,
                      int32_t mid_row, const CsrHints& hints, hipStream_t s, const UpdateArgs* upd)
{
    // a mask that no kernel of the launch looks at must not pass for one that was applied
    if (a.x_mask && (upd || !csr_mask_usable(a, hints))) return hipErrorInvalidValue;
    const bool narrow = upd ? fused_narrow(a) : !a.rowend && narrow_rows(a, hints);
    CsrShape sh = pick_shape(a, narrow);
    // the other forms address indices and values, too, with 32-bit offsets from a uniform base: short rows are bound by the vector units as much as by
    // their chains (communities, 131,072 rows of 20, fp32, 32 columns: 21.4 -> 20.4 us; with no instructions spent on an activation that is not asked
    // for, and the halves of a group added in one each, bf16, 64 columns: 23.8 -> 22.9)
    if (hints.entries > ((int64_t)1 << 30)) sh.wide = true;
    CsrWork wk{};
    wk.n_segs = n_segs; wk.segs = segs; wk.partial = partial; wk.n_mid = n_mid; wk.mid_rows = mid_rows;
    wk.n_items = n_items; wk.row_list = row_list; wk.route = route; wk.mid_row = mid_row;
    // vector stores need Y rows aligned for what a lane stores at once (16-bit results leave in pieces of up to 8 bytes)
    const int yv = sh.vec < 4 ? sh.vec : 4;
    wk.y_vec = a.ldy % yv == 0 && (uintptr_t)a.Y % (yv * (a.y_dtype == HCSPMM_F32 ? 4 : 2)) == 0;
    wk.skip_empty = a.acc && !a.relu && (const void*)a.acc == (const void*)a.Y && a.ldacc == a.ldy && a.y_dtype == HCSPMM_F32;
    int run = 5;
    if (tune().xcd_chunk >= 0) for (run = -1; tune().xcd_chunk >> (run + 1);) ++run;
    if (upd) {
        // one slice, and a row per group whatever the matrix
        wk.grid = csr_grid(n_segs, n_mid, n_items, a.d, 1, a.d, run, sh.group);
        if (wk.grid.rows_per_group > 1) return hipErrorInvalidValue;        // (update_fusable bounds the rows)
        if (wk.grid.blocks() <= 0) return hipSuccess;
#define HC_LAUNCH_CSRF(XK, V, NVV, L, GR, W) hipLaunchKernelGGL((k_csr_fused<Gather<XK, V, NVV, L, GR, W>>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a, *upd)
        HC_CSR_DISPATCH(HC_LAUNCH_CSRF)
#undef HC_LAUNCH_CSRF
        return hipGetLastError();
    }
    int32_t slice_w = a.d;
    const int n_slices = pick_slices(a, hints, slice_w);
    // On the smallest matrices every row is a mid row: its non-zeros are spread over four groups instead of queueing in one
    // (2,708 nodes, 32 columns: 5.6 -> 3.6 us of kernel time).  From half of the chip's waves on (256 CUs x 32) starting them
    // costs more than the shorter chains save (a group / a wave per row, us, fp32: 2,000 rows of 11, 96 columns: 6.7 / 5.1;
    // 3,000 of 21, 160 columns in two slices: 7.8 / 10.3; communities of 20, 7,936 rows, 128 columns: 7.4 / 11.1; bf16, 128
    // columns: 4,000 of 11: 6.6 / 5.9; 6,000 of 13: 7.1 / 6.7; 8,000 of 31: 8.1 / 8.9).
    const bool few_rows = n_items > 0 && few_rows_form(a, n_slices);
    if (few_rows) {
        wk.n_mid = a.n_rows;
        wk.mid_rows = nullptr;
        wk.mid_row = hints.long_row;
        wk.n_items = 0;
    }
    wk.grid = csr_grid(n_segs, wk.n_mid, wk.n_items, a.d, n_slices, slice_w, run, sh.group, tune().rpg >= 1 && tune().rpg <= sh.group ? tune().rpg : 1);
    if (wk.grid.blocks() <= 0) return hipSuccess;
    if (wk.grid.rows_per_group > 1) sh.wide = true;
    if (wk.grid.n_slices > 1) {
        SpmmArgs t = a;
        t.d = wk.grid.slice_w;
        const bool wide = sh.wide;
        sh = pick_shape(t, false);
        sh.wide = wide;
    }
#define HC_LAUNCH_CSR(XK, V, NVV, L, GR, W) hipLaunchKernelGGL((k_csr<Gather<XK, V, NVV, L, GR, W>>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a)
#define HC_LAUNCH_PANEL(XK, V, NVV, L, GR, W) hipLaunchKernelGGL((k_csr<Gather<XK, V, NVV, L, GR, W, true>>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a)
    const int most = few_waves(a, hints, sh, wk.grid.n_slices > 1 ? wk.grid.slice_w : a.d);
#define HC_LAUNCH_FEW(XK, V, NVV, L, GR, W)                                                                                                     \
    if (most == 2) hipLaunchKernelGGL((k_csr_few<Gather<XK, V, NVV, L, GR, W>, 2>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a); \
    else hipLaunchKernelGGL((k_csr_few<Gather<XK, V, NVV, L, GR, W>, 3>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a)
#define HC_LAUNCH_FEW_PANEL(XK, V, NVV, L, GR, W)                                                                                                     \
    if (most == 2) hipLaunchKernelGGL((k_csr_few<Gather<XK, V, NVV, L, GR, W, true>, 2>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a); \
    else hipLaunchKernelGGL((k_csr_few<Gather<XK, V, NVV, L, GR, W, true>, 3>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a)
    if (a.x_mask) {
        // (what csr_mask_usable has found, once more where the launch is chosen)
        if (most != 0 || sh.wide || sh.vec != 4 || sh.lanes != 16 || sh.group != 16 || sh.nv > 2 || few_rows ||
            (wk.grid.n_slices > 1 && wk.grid.slice_w % 64 != 0)) return hipErrorInvalidValue;
        if (sh.nv == 1) hipLaunchKernelGGL((k_csr<Gather<0, 4, 1, 16, 16, false, false, true>>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a);
        else hipLaunchKernelGGL((k_csr<Gather<0, 4, 2, 16, 16, false, false, true>>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a);
        return hipGetLastError();
    }
    if (a.rowend) {
        // panels are taken for rows of kPanelRowBytes and more: 16-byte vectors, two per lane at most (wider slices take turns)
        if (sh.vec != (a.x_dtype == HCSPMM_F32 ? 4 : 8)) return hipErrorInvalidValue;
        if (most > 0) {
            if (a.x_dtype == HCSPMM_BF16) HC_CSR_ONE(HC_LAUNCH_FEW_PANEL, 1, 8, 2, 16, 16);
            else HC_CSR_ONE(HC_LAUNCH_FEW_PANEL, 2, 8, 2, 16, 16);
        } else if (a.x_dtype == HCSPMM_F32) { HC_CSR_PANEL_DISPATCH(HC_LAUNCH_PANEL, 0, 4) }
        else if (a.x_dtype == HCSPMM_BF16) { HC_CSR_PANEL_DISPATCH(HC_LAUNCH_PANEL, 1, 8) }
        else { HC_CSR_PANEL_DISPATCH(HC_LAUNCH_PANEL, 2, 8) }
        return hipGetLastError();
    }
    if (few_rows && most == 0 && !sh.wide && !route && !a.acc && a.ldx <= INT32_MAX && a.ldy <= INT32_MAX && wk.grid.n_slices <= 255) {
        const CsrFewRows r{a.rowptr, a.colind, a.vals, a.X, a.Y, segs, partial, (int32_t)a.ldx, (int32_t)a.ldy, a.n_rows, a.d, wk.mid_row, n_segs,
                           wk.grid.seg_blocks, wk.grid.mid_blocks, wk.grid.run_mid, wk.grid.slice_w, (uint8_t)wk.grid.n_slices, (uint8_t)a.y_dtype,
                           (uint8_t)(a.relu != 0), (uint8_t)wk.y_vec};
#define HC_LAUNCH_FEW_ROWS(XK, V, NVV, L, GR, W) hipLaunchKernelGGL((k_csr_few_rows<Gather<XK, V, NVV, L, GR, false>>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, r)
        HC_CSR_DISPATCH(HC_LAUNCH_FEW_ROWS)
#undef HC_LAUNCH_FEW_ROWS
        return hipGetLastError();
    }
    if (most > 3) {
#define HC_LAUNCH_SOME(XK, V, L, MOST) hipLaunchKernelGGL((k_csr_few<Gather<XK, V, 1, L, 16, false>, MOST>), dim3((unsigned)wk.grid.blocks()), dim3(256), 0, s, wk, a)
#define HC_LAUNCH_SOME_OF(XK, V)                                                                          \
    if (sh.lanes == 8) { if (most == 4) HC_LAUNCH_SOME(XK, V, 8, 4); else HC_LAUNCH_SOME(XK, V, 8, 5); } \
    else if (most == 4) HC_LAUNCH_SOME(XK, V, 16, 4);                                                    \
    else HC_LAUNCH_SOME(XK, V, 16, 5)
        if (a.x_dtype == HCSPMM_F32) { HC_LAUNCH_SOME_OF(0, 4); }
        else if (a.x_dtype == HCSPMM_BF16) { HC_LAUNCH_SOME_OF(1, 8); }
        else { HC_LAUNCH_SOME_OF(2, 8); }
#undef HC_LAUNCH_SOME_OF
#undef HC_LAUNCH_SOME
        return hipGetLastError();
    }
    if (most > 0) {
        if (a.x_dtype == HCSPMM_F32) HC_CSR_ONE(HC_LAUNCH_FEW, 0, 4, 4, 16, 16);
        else if (a.x_dtype == HCSPMM_BF16) HC_CSR_ONE(HC_LAUNCH_FEW, 1, 8, 2, 16, 16);
        else HC_CSR_ONE(HC_LAUNCH_FEW, 2, 8, 2, 16, 16);
        return hipGetLastError();
    }
    HC_CSR_DISPATCH(HC_LAUNCH_CSR)
#undef HC_LAUNCH_FEW_PANEL
#undef HC_LAUNCH_FEW
#undef HC_LAUNCH_PANEL
#undef HC_LAUNCH_CSR
    return hipGetLastError();
}

hipError_t launch_update_rest(const SpmmArgs& a, int32_t n_rest, const int32_t* rest_rows, const UpdateArgs& upd,
                              hipStream_t s)
{
    if (n_rest <= 0) return hipSuccess;
    // several consecutive tiles per wave once there are enough tiles to keep every CU supplied with waves
    const int64_t n_tiles = ((int64_t)n_rest + 15) / 16;
    int tpw = 1;
    while (tpw < 8 && n_tiles / (2 * tpw) >= 16384) tpw *= 2;
    if (tune().tiles_per_wave >= 1 && tune().tiles_per_wave <= 64) tpw = tune().tiles_per_wave;
    const dim3 grid((unsigned)((n_tiles + 4 * (int64_t)tpw - 1) / (4 * (int64_t)tpw)));
    const int nt = update_tile_nt(upd, 1);
#define HC_REST(ZD)                                                                                                   \
    {                                                                                                                 \
        if (nt == 4) hipLaunchKernelGGL((k_update_rest<ZD, 4>), grid, dim3(256), 0, s, n_rest, rest_rows, tpw, a, upd);      \
        else if (nt == 2) hipLaunchKernelGGL((k_update_rest<ZD, 2>), grid, dim3(256), 0, s, n_rest, rest_rows, tpw, a, upd); \
        else hipLaunchKernelGGL((k_update_rest<ZD, 1>), grid, dim3(256), 0, s, n_rest, rest_rows, tpw, a, upd);              \
    }
    if (a.d <= 64) HC_REST(64)
    else if (a.d <= 128) HC_REST(128)
    else if (a.d <= 256) HC_REST(256)
    else return hipErrorInvalidValue;
#undef HC_REST
    return hipGetLastError();
}

// ---- measurement aid: the bare gather ------------------------------------------------------------
// Reads row index[i] of X for every i and does nothing else a sparse product would do (no row
// structure, no values, no output rows): a lane group takes a contiguous run of indices, 16 at a
// time with one coalesced load, keeps as many row requests in flight as the scalar path, and adds
// what arrives into registers; one vector per lane is stored at the end so the loads stay live.
// Its duration is what the scalar path's loop takes for the gather alone of the same stream.
template <class G>
__global__ __launch_bounds__(256) void k_probe_gather(const int32_t* __restrict__ index, int64_t n, int64_t per_group,
                                                      SpmmArgs a, int32_t n_rows_x, float* __restrict__ out)
{
    // workgroups in XCD-local runs of 32, like the scalar path's short rows (the grid is padded to whole rounds)
    const int64_t x = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int64_t blk = ((q / 32) * 8 + x) * 32 + q % 32;
    const int64_t grp = blk * (256 / G::GROUP) + threadIdx.x / G::GROUP;
    const int lig = threadIdx.x % G::GROUP;
    const int64_t b = min(n, grp * per_group), e = min(n, b + per_group);
    G g;
    g.init(a, 0, a.d, lig);
    float acc[G::N];
    vzero(acc);
    for (int64_t k0 = b; k0 < e; k0 += G::GROUP) {                // (a group past the end of the stream has b == e)
        const int64_t k = min(k0 + lig, e - 1);
        const int32_t c = min(max(index[k], 0), n_rows_x - 1);  // whatever the stream holds, the read stays inside X
        g.batch(g.key(c), 1.f, (int)min((int64_t)G::GROUP, e - k0), acc, [] {});
    }
    float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < G::N; ++i) t[i & 3] += acc[i];
    *reinterpret_cast<float4*>(out + ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4) = make_float4(t[0], t[1], t[2], t[3]);
}

constexpr int kProbeGroup = 16;
// Launch shape of the probe: indices per lane group 512 (long enough to amortise the start-up) unless the stream is too
// short to give every CU some tens of workgroups that way -- then fewer, down to 64.
static void probe_gather_shape(int64_t n, int64_t& per_group, int64_t& blocks)
{
    const int64_t groups_per_block = 256 / kProbeGroup;
    per_group = (n / (8192 * groups_per_block) + 63) / 64 * 64;
    per_group = per_group < 64 ? 64 : (per_group > 512 ? 512 : per_group);
    const int64_t groups = (n + per_group - 1) / per_group;
    blocks = (groups + groups_per_block - 1) / groups_per_block;
    blocks = (blocks + 255) / 256 * 256;                       // whole rounds of eight XCD-local runs of 32 workgroups
}

int64_t probe_gather_blocks(int64_t n, int32_t d)
{
    (void)d;
    int64_t per_group, blocks;
    probe_gather_shape(n, per_group, blocks);
    return blocks;
}

hipError_t launch_probe_gather(const int32_t* index, int64_t n, const float* X, int64_t ldx, int32_t d, int32_t n_rows_x,
                               float* out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t per_group, blocks;
    probe_gather_shape(n, per_group, blocks);
    SpmmArgs a{};
    a.n_cols = n_rows_x; a.X = X; a.ldx = ldx; a.d = d; a.x_dtype = HCSPMM_F32;
    const CsrShape sh = pick_shape(a, false);
#define HC_PROBE(XK, V, NVV, L, GR, W) hipLaunchKernelGGL((k_probe_gather<Gather<XK, V, NVV, L, GR, W>>), dim3((unsigned)blocks), dim3(256), 0, s, index, n, per_group, a, n_rows_x, out)
    HC_CSR_DISPATCH32_16(HC_PROBE)
#undef HC_PROBE
    return hipGetLastError();
}

hipError_t launch_reduce_partials(const SpmmArgs& a, int32_t n_multi, const MultiRow* multi, const float* partial,
                                  hipStream_t s)
{
    if (n_multi <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce_partials, dim3(n_multi), dim3(256), 0, s, n_multi, multi, partial, a);
    return hipGetLastError();
}

}  // namespace hcspmm
