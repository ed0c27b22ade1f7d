// Store and query preparation: unit-normalise raw hidden-state rows and
// round them to bf16 (Sec. 4 (i), Eq. 1: keys are kept L2-normalised in half
// precision; queries get the same treatment so that the dot product of the
// two operands is their cosine, Algorithm 1 retrieve step).
//
// Small calls (queries, the positions of a step): one 1024-thread block per
// row (a row of up to 8192 columns is read once, at most eight values per
// thread: the latency of one row's work, not memory, sets the time).  Bulk
// appends: store_rows_kernel, eight rows per workgroup.  The squared norm is
// accumulated in double, each quotient by it rounded once (RowScale: nearly
// all of them without a division), so identical raw rows always produce
// identical stored bits, wherever they sit in the pool and whichever of the
// kernels took them: where the last bits of the norm decide a value, the bulk
// kernel sums the squares again in the one-row kernels' order.
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "rowops.hpp"

namespace oil {

// Destination layouts of a normalised row (offsets in bf16 elements; row i,
// column j; ld = width rounded up to 64):
//   kLayoutRows: i * ld + j (queries of the GEMV scan).
//   kLayoutTiled: rows in blocks of 32, columns in windows of 64; each
//     (row block, window) pair is a 4 KiB tile in MFMA operand order, tile
//     (i / 32, j / 64) starting at (i / 32) * rs + (j / 64) * ws:
//       (i / 32) * rs + (j / 64) * ws + (s * 64 + lane) * 8 + e,
//     s = (j % 32) / 8, e = j % 8, lane = i % 32 + 32 * ((j % 64) / 32).
//     One 16-byte load per lane of a tile sub-step s reads 1 KiB contiguous.
//     The key pool uses it, and so do the MFMA scan's query fragments
//     (rs = 2048, ws = 2048 * query tiles).
__device__ __forceinline__ int64_t layout_offset(int layout, int64_t i, int32_t j, int32_t ld,
                                                 int64_t rs, int64_t ws)
{
    if (layout == kLayoutRows)
        return i * (int64_t)ld + j;
    const int s = (j >> 3) & 3, e = j & 7;
    const int lane = (int)(i & 31) + 32 * ((j >> 5) & 1);
    return (i >> 5) * rs + (int64_t)(j >> 6) * ws + (s * 64 + lane) * 8 + e;
}

constexpr int kRowThreads = 1024;

__global__ __launch_bounds__(kRowThreads) void normalize_rows_kernel(
    const void* __restrict__ raw, int dtype, int32_t d, int64_t n_rows_in, uint16_t* __restrict__ out,
    int64_t row_offset, int32_t ld, int layout, int64_t rs, int64_t ws, const int32_t* __restrict__ tok_in,
    const int32_t* __restrict__ trace_in, const int32_t* __restrict__ prompt_in,
    int32_t* __restrict__ tok_out, int32_t* __restrict__ trace_out, int32_t* __restrict__ prompt_out)
{
    __shared__ double red[kRowThreads / 64];
    const int64_t r = blockIdx.x;  // row within this call
    const bool live = r < n_rows_in;
    const int64_t dst_row = row_offset + r;
    normalize_row<kRowThreads>(raw, dtype, r, d, ld, live, red, [&](int32_t j, uint16_t bits) {
        out[layout_offset(layout, dst_row, j, ld, rs, ws)] = bits;
    });
    if (threadIdx.x == 0 && live && tok_out) {
        tok_out[dst_row] = tok_in[r];
        trace_out[dst_row] = trace_in[r];
        if (prompt_out)
            prompt_out[dst_row] = prompt_in[r];
    }
}

// Nearest OCP E4M3 code of v (|v| <= 448: larger magnitudes saturate to
// 448), ties to the even code.  The representable magnitudes are multiples of
// 2^(E - 3) in [2^E, 2^(E + 1)) for E >= -6 and of 2^-9 below 2^-6; scaling by
// the spacing is exact, so one rint (nearest-even) does the rounding.  The
// multiple r lands in [8, 16] (16 carries into the next binade) or, below
// 2^-6, in [0, 8]; either way the code's low 7 bits are ((E + 7) << 3) + r - 8
// or r.
__device__ __forceinline__ uint8_t double_to_e4m3_rne(double v)
{
    const uint8_t sign = __double_as_longlong(v) < 0 ? 0x80 : 0;
    const double a = fabs(v);
    if (!(a < 448.0))
        return (uint8_t)(sign | 0x7E);
    if (a >= 0x1p-6) {
        const int E = ilogb(a);
        const double r = rint(ldexp(a, 3 - E));
        return (uint8_t)(sign | (uint8_t)(((E + 7) << 3) + (int)r - 8));
    }
    return (uint8_t)(sign | (uint8_t)rint(ldexp(a, 9)));
}

// |q| in multiples of the spacing of E4M3 codes around it (exact; in [0, 16]),
// and what to add to the rounded multiple for the code of that binade.
__device__ __forceinline__ float e4m3_steps(float q, float& scale, int& base)
{
    const int E = max((int)((__float_as_uint(q) >> 23) & 255u), 127 - 6);  // biased exponent, at least that of 2^-6
    scale = __uint_as_float((uint32_t)(127 + 127 + 3 - E) << 23);
    base = ((E - 120) << 3) - 8;
    return fabsf(q) * scale;
}

// Whether the scaled quotient q is too close to the middle of two E4M3 codes
// for its float bits to decide the rounding: within four ulps of a middle, or
// below 2^-6, where the codes' spacing no longer follows q's exponent (about
// one value in 4,000 of a Gaussian row).
__device__ __forceinline__ bool e4m3_near(float q)
{
    const uint32_t u = __float_as_uint(q);
    return ((u - 0x7FFFCu) & 0xFFFFFu) <= 8u || (u << 1) - 1u < 2u * 0x3C800000u - 1u;
}

// The code that the scaled quotient v / norm * 2^shift rounds to, for q =
// v * s.inv with s already scaled by 2^shift (its norm is not) and a near
// number of steps.  divided: set where the last bits of s.norm decide.
__device__ __forceinline__ uint8_t e4m3_settle(float v, float q, const RowScale& s, int shift, bool& divided)
{
    float scale;
    int base;
    const float a = e4m3_steps(q, scale, base), low = floorf(a);
    const float rest = quotient_rest(v, q, s) * scale;
    const float above = (a - (low + 0.5f)) + (q < 0.f ? -rest : rest);
    if (!s.fast || !(fabsf(above) > a * 0x1p-40f)) {
        divided = true;
        return double_to_e4m3_rne(ldexp((double)v / s.norm, shift));
    }
    return (uint8_t)(((__float_as_uint(q) >> 24) & 0x80u) |
                     (uint32_t)(base + (int)low + (above > 0.f ? 1 : 0)));
}

// s scaled for fp8 rows: inv and inv_lo times 2^shift (exact).
__device__ __forceinline__ RowScale scaled(RowScale s, int shift)
{
    s.inv = ldexpf(s.inv, shift);
    s.inv_lo = ldexpf(s.inv_lo, shift);
    return s;
}

__device__ __forceinline__ uint8_t unit_e4m3(float v, const RowScale& s, int shift, bool& divided)
{
    const float q = v * s.inv;
    if (!s.fast || e4m3_near(q))
        return e4m3_settle(v, q, s, shift, divided);
    return (uint8_t)__builtin_amdgcn_cvt_pk_fp8_f32(q, q, 0, false);
}

// fp8 tile layout (bytes): rows in blocks of 32, columns in windows of 128;
// each (row block, window) pair is a 4 KiB tile, one 16-byte load per lane
// and sub-step p (lane i % 32 + 32 h holds row i % 32), two sub-steps per
// fp8 MFMA operand (keys and query fragments share the layout, so an
// operand slot holds the same column for both):
//   (i / 32) * rs + (j / 128) * ws + (p * 64 + lane) * 16 + hh * 8 + e,
//   s = (j % 128) / 16, p = s / 2, hh = s % 2, e = j % 8,
//   lane = i % 32 + 32 * ((j % 16) / 8).
__device__ __forceinline__ int64_t fp8_offset(int64_t i, int32_t j, int64_t rs, int64_t ws)
{
    const int jw = j & 127, s = jw >> 4, p = s >> 1, hh = s & 1, e = jw & 7;
    const int lane = (int)(i & 31) + 32 * ((jw >> 3) & 1);
    return (i >> 5) * rs + (int64_t)(j >> 7) * ws + (p * 64 + lane) * 16 + hh * 8 + e;
}

// Block-wide maximum of one non-negative double per thread of an NT-thread
// block (red: NT / 64 doubles).
template <int NT>
__device__ __forceinline__ double block_max(double m, double* red)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        m = fmax(m, __shfl_xor(m, o, kWave));
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = m;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int w = 1; w < NT / 64; w++)
        t = fmax(t, red[w]);
    return t;
}

// Power-of-two scale shift putting the row's largest magnitude m in [128, 256).
__device__ __forceinline__ int fp8_shift(double m) { return m > 0.0 ? 7 - ilogb(m) : 0; }

// Whether m is so near a power of two (2^-40 of it, on either side) that the last
// bits of the norm decide it: its mantissa is within 2^12 steps above zero, or
// 2^13 below the next binade's.  (Working out both neighbours' exponents: 20,000
// bf16 rows of 1,000 / 5,120 columns 22.0 / 61.8 us against 21.5 / 61.0.)
__device__ __forceinline__ bool fp8_shift_near(double m)
{
    const uint64_t u = (uint64_t)__double_as_longlong(m) + (1u << 13);
    return m > 0.0 && (u & ((1ull << 52) - 1)) <= 3u << 12;
}

// One row of quantize_rows_kernel for ld8 <= NT * NV, read once into
// registers; the same arithmetic as the general path.  Returns the shift.
template <int NT, int NV, class Dst>
__device__ __forceinline__ int quantize_row_regs(const void* raw, int dtype, int64_t r, int32_t d, int32_t ld8,
                                                 bool live, double* red, Dst dst)
{
    const int t = threadIdx.x;
    float v[NV];
    load_row<NT, NV>(raw, dtype, r, d, live, v);
    const RowScale sc = row_scale(sqrt(block_sum<NT>(sum_squares(v), red)));
    // division is monotonic: the largest quotient is the largest value's
    float top = 0.f;
#pragma unroll
    for (int i = 0; i < NV; i++)
        top = fmaxf(top, fabsf(v[i]));
    const int shift = fp8_shift(block_max<NT>(sc.norm > 0.0 ? (double)top / sc.norm : 0.0, red));
    const RowScale s8 = scaled(sc, shift);
    bool divided;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int32_t j = i * NT + t;
        if (j < ld8)
            dst(j, (j < d && sc.norm > 0.0) ? unit_e4m3(v[i], s8, shift, divided) : (uint8_t)0);
    }
    return shift;
}

__global__ __launch_bounds__(kRowThreads) void quantize_rows_kernel(
    const void* __restrict__ raw, int dtype, int32_t d, int64_t n_rows_in, uint8_t* __restrict__ out,
    int64_t row_offset, int32_t ld8, int64_t rs, int64_t ws, float* __restrict__ inv_scale,
    const int32_t* __restrict__ tok_in, const int32_t* __restrict__ trace_in,
    const int32_t* __restrict__ prompt_in, int32_t* __restrict__ tok_out, int32_t* __restrict__ trace_out,
    int32_t* __restrict__ prompt_out)
{
    constexpr int NT = kRowThreads;
    __shared__ double red[NT / 64];
    const int64_t r = blockIdx.x;
    const bool live = r < n_rows_in;
    const int64_t dst_row = row_offset + r;
    const int t = threadIdx.x;
    const auto put = [&](int32_t j, uint8_t c) {
        out[rs > 0 ? fp8_offset(dst_row, j, rs, ws) : dst_row * ld8 + j] = c;
    };
    int shift;
    if (ld8 <= NT * 4) {
        shift = quantize_row_regs<NT, 4>(raw, dtype, r, d, ld8, live, red, put);
    } else if (ld8 <= NT * 8) {
        shift = quantize_row_regs<NT, 8>(raw, dtype, r, d, ld8, live, red, put);
    } else {
        // the unit row in double, exactly as the bf16 store computes it
        double ss = 0.0;
        if (live)
            for (int32_t j = t; j < d; j += NT) {
                const double x = load_raw(raw, dtype, r * d + j);
                ss += x * x;
            }
        const double norm = sqrt(block_sum<NT>(ss, red));
        double m = 0.0;
        if (live && norm > 0.0)
            for (int32_t j = t; j < d; j += NT)
                m = fmax(m, fabs(load_raw(raw, dtype, r * d + j) / norm));
        shift = fp8_shift(block_max<NT>(m, red));
        for (int32_t j = t; j < ld8; j += NT) {
            uint8_t c = 0;
            if (live && j < d && norm > 0.0)
                c = double_to_e4m3_rne(ldexp(load_raw(raw, dtype, r * d + j) / norm, shift));
            put(j, c);
        }
    }
    if (t == 0) {
        inv_scale[dst_row] = live ? ldexpf(1.f, -shift) : 1.f;
        if (live && tok_out) {
            tok_out[dst_row] = tok_in[r];
            trace_out[dst_row] = trace_in[r];
            if (prompt_out)
                prompt_out[dst_row] = prompt_in[r];
        }
    }
}

// ----------------------------------------------------------------- bulk appends
// One 512-thread workgroup per R = 8 (or 4) stored rows, aligned to R, so they
// share a 32-row block.  Lane l of a wave holds row l % R; the 64 / R lanes of
// a row take neighbouring 8-column chunks (fp8: 16 columns), so a wave's loads
// read contiguous stretches of each row and its stores write 16 bytes per
// lane, 16 R contiguous bytes of the tile per R rows.  (One workgroup per row
// stored two bytes per thread, scattered over the tiles, and rounded every
// value through a division in double.)
// The rows stay in registers between the norm and the rounding: memory is
// read once and written once, which is what bounds it: 60,001 rows of 4,096
// bf16 values into a bf16 pool 896 -> 190 us (5.2 TB/s in and out), 20,011 rows
// of 5,120 f32 values into an fp8 pool 331 -> 119 (4.3 TB/s).
//
// VEC: whole 16-byte pieces of every row are aligned (base and row stride);
// other widths load element by element.
constexpr int kBulkThreads = 512;

// The 16 codes of two chunks of a unit row scaled by 2^shift (s is scaled), and
// whether some of them need settling (settle_e4m3_16).
template <bool F32>
__device__ __forceinline__ u32x4 unit_e4m3_16(const u32x4 (&x)[2][F32 ? 2 : 1], const RowScale& s, bool& near)
{
    u32x4 w = {0, 0, 0, 0};
    near = !s.fast;
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
        const float q0 = chunk_value<F32>(x[e >> 3], e & 7) * s.inv;
        const float q1 = chunk_value<F32>(x[e >> 3], (e & 7) + 1) * s.inv;
        near |= e4m3_near(q0) || e4m3_near(q1);
        if (e & 2)
            w[e >> 2] = __builtin_amdgcn_cvt_pk_fp8_f32(q0, q1, w[e >> 2], true);
        else
            w[e >> 2] = __builtin_amdgcn_cvt_pk_fp8_f32(q0, q1, w[e >> 2], false);
    }
    return w;
}

// The same with every value settled (zeros for a zero or NaN row).
template <bool F32>
__device__ __forceinline__ u32x4 settle_e4m3_16(const u32x4 (&x)[2][F32 ? 2 : 1], const RowScale& s, int shift,
                                                bool& divided)
{
    u32x4 w = {0, 0, 0, 0};
    if (!(s.norm > 0.0))
        return w;
    for (int e = 0; e < 16; e++) {  // rolled: one copy of the division in double
        float v = 0.f;
#pragma unroll
        for (int f = 0; f < 16; f++)
            v = f == e ? chunk_value<F32>(x[f >> 3], f & 7) : v;
        const uint32_t bits = (uint32_t)unit_e4m3(v, s, shift, divided) << ((e & 3) * 8);
#pragma unroll
        for (int q = 0; q < 4; q++)
            w[q] |= q == (e >> 2) ? bits : 0u;
    }
    return w;
}

// Wavefronts per SIMD that the registers must leave room for: three workgroups
// per compute unit where a thread's raw values fit 40 registers, else two.
constexpr int bulk_waves(int fmt, bool f32, bool vec, int ni)
{
    return vec && ni * (fmt == kKeyFp8 ? 2 : 1) * (f32 ? 8 : 4) <= 40 ? 6 : 4;
}

template <int FMT, bool F32, bool VEC, int NI, int R>
__global__ __launch_bounds__(kBulkThreads) __attribute__((amdgpu_waves_per_eu(bulk_waves(FMT, F32, VEC, NI)))) void
store_rows_kernel(
    const void* __restrict__ raw, int32_t d, int64_t n, uint8_t* __restrict__ out, int64_t row_offset, int32_t ld,
    int64_t rs, int64_t ws, float* __restrict__ inv_scale, const int32_t* __restrict__ tok_in,
    const int32_t* __restrict__ trace_in, const int32_t* __restrict__ prompt_in, int32_t* __restrict__ tok_out,
    int32_t* __restrict__ trace_out, int32_t* __restrict__ prompt_out)
{
    constexpr int H = FMT == kKeyFp8 ? 2 : 1;  // 8-column chunks per unit
    constexpr int kUnits = kBulkThreads / R;     // units of a row per iteration
    __shared__ double red[kBulkThreads / 64][R];
    __shared__ float redm[kBulkThreads / 64][R];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & (R - 1);
    const int u0 = wave * (64 / R) + lane / R;
    const int64_t dst = (row_offset / R + blockIdx.x) * R + r;
    const int64_t src = dst - row_offset;
    const bool live = src >= 0 && src < n;
    const int64_t at = (live ? src : 0) * d;  // rows outside the call read row 0 and store nothing
    const int units = ld / (8 * H);
    // first column of chunk h of unit u
    auto col_of = [&](int u, int h) -> int32_t {
        if constexpr (FMT == kKeyFp8)
            return (u >> 3) * 128 + ((u & 7) >> 1) * 32 + (u & 1) * 8 + h * 16;
        else
            return u * 8;
    };
    u32x4 x[NI][H][F32 ? 2 : 1];
#pragma unroll
    for (int i = 0; i < NI; i++)
#pragma unroll
        for (int h = 0; h < H; h++)
            load_chunk<F32, VEC>(raw, at, col_of(u0 + i * kUnits, h), d, x[i][h]);
    auto value = [&](int i, int h, int e) { return chunk_value<F32>(x[i][h], e); };
    double ss = 0.0;
    float top = 0.f;
#pragma unroll
    for (int i = 0; i < NI; i++)
#pragma unroll
        for (int h = 0; h < H; h++)
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const float v = value(i, h, e);
                const double vd = v;
                ss += vd * vd;
                if constexpr (FMT == kKeyFp8)
                    top = fmaxf(top, fabsf(v));
            }
#pragma unroll
    for (int o = 32; o >= R; o >>= 1) {
        ss += __shfl_xor(ss, o, kWave);
        if constexpr (FMT == kKeyFp8)
            top = fmaxf(top, __shfl_xor(top, o, kWave));
    }
    if (lane < R) {
        red[wave][lane] = ss;
        if constexpr (FMT == kKeyFp8)
            redm[wave][lane] = top;
    }
    __syncthreads();
    ss = 0.0;
#pragma unroll
    for (int w = 0; w < kBulkThreads / 64; w++) {
        ss += red[w][r];
        if constexpr (FMT == kKeyFp8)
            top = fmaxf(top, redm[w][r]);
    }
    if constexpr (!F32) {
        // unpacked again below: the floats of the norm would otherwise stay in
        // registers beside the raw pieces (half the workgroups in flight)
#pragma unroll
        for (int i = 0; i < NI; i++)
#pragma unroll
            for (int h = 0; h < H; h++)
                asm volatile("" : "+v"(x[i][h][0]));
    }
    RowScale sc = row_scale(sqrt(ss));
    int shift = 0;
    if constexpr (FMT == kKeyFp8) {
        const auto largest = [&] { return sc.norm > 0.0 ? (double)top / sc.norm : 0.0; };
        const bool near = live && fp8_shift_near(largest());
        if (__any(near))
            column_order_norms<kRowThreads, F32, R>(near, raw, at, d, sc.norm);
        shift = fp8_shift(largest());
        sc = scaled(sc, shift);
    }
    uint8_t* base = out + (dst >> 5) * rs;
    const int row32 = (int)(dst & 31);
    auto put = [&](int i, const u32x4& w) {
        const int u = u0 + i * kUnits;
        // 16-byte slot of (row, unit) in its 4 KiB tile
        const int slot = FMT == kKeyFp8 ? ((u & 7) >> 1) * 64 + row32 + 32 * (u & 1)
                                        : (u & 3) * 64 + row32 + 32 * ((u & 7) >> 2);
        __builtin_nontemporal_store(w, (u32x4*)(base + (int64_t)(u >> 3) * ws + slot * 16));
    };
    // the decided units first; the few others are then settled and stored again
    uint32_t open = 0;
#pragma unroll
    for (int i = 0; i < NI; i++) {
        if (!live || u0 + i * kUnits >= units)
            break;
        bool near;
        u32x4 w;
        if constexpr (FMT == kKeyFp8)
            w = unit_e4m3_16<F32>(x[i], sc, near);
        else
            w = unit_chunk_bf16<F32>(x[i][0], sc, near);
        put(i, w);
        open |= near ? 1u << i : 0u;
    }
    auto settle = [&](int i, const u32x4(&y)[H][F32 ? 2 : 1]) -> bool {
        bool divided = false;
        if constexpr (FMT == kKeyFp8)
            put(i, settle_e4m3_16<F32>(y, sc, shift, divided));
        else
            put(i, settle_chunk_bf16<F32>(y[0], sc, divided));
        return divided;
    };
    uint32_t divided = 0;  // units with a value that the norm's last bits decide
    while (open) {
        const int i = __ffs((int)open) - 1;
        open &= open - 1;
        u32x4 y[H][F32 ? 2 : 1];
#pragma unroll
        for (int h = 0; h < H; h++)
#pragma unroll
            for (int p = 0; p < (F32 ? 2 : 1); p++) {
                y[h][p] = x[0][h][p];
#pragma unroll
                for (int j = 1; j < NI; j++)
                    y[h][p] = j == i ? x[j][h][p] : y[h][p];
            }
        divided |= settle(i, y) ? 1u << i : 0u;
    }
    if (__any(divided)) {
        // (the row's place is worked out again, and the row read again, so that
        // no register holds them until here)
        int64_t first = row_offset;
        asm volatile("" : "+s"(first));
        const int64_t src2 = (first / R + blockIdx.x) * R + r - first;
        const int64_t at2 = (src2 >= 0 && src2 < n ? src2 : 0) * d;
        column_order_norms<kRowThreads, F32, R>(divided != 0, raw, at2, d, sc.norm);
        while (divided) {
            const int i = __ffs((int)divided) - 1;
            divided &= divided - 1;
            u32x4 y[H][F32 ? 2 : 1];
#pragma unroll
            for (int h = 0; h < H; h++)
                load_chunk<F32, VEC>(raw, at2, col_of(u0 + i * kUnits, h), d, y[h]);
            settle(i, y);
        }
    }
    if (live && u0 == 0) {  // one lane per row
        if constexpr (FMT == kKeyFp8)
            inv_scale[dst] = ldexpf(1.f, -shift);
        tok_out[dst] = tok_in[src];
        trace_out[dst] = trace_in[src];
        if (prompt_out)
            prompt_out[dst] = prompt_in[src];
    }
}

// Rows from which a call into tiles takes store_rows_kernel: below, a
// 1024-thread workgroup per row fills the chip sooner (512 rows of 8,192 bf16
// columns 16.6 us against 18.3; 768 rows 22.8 against 19.1, 2,048 rows of
// 4,096 31 against 14).
#ifndef OIL_BULK_MIN
#define OIL_BULK_MIN 640
#endif
static bool bulk_rows(int64_t n, int32_t ld) { return n >= OIL_BULK_MIN && ld <= 8192; }

// rs, ws: tile strides in bytes.
template <int FMT>
static hipError_t launch_store_rows(const void* raw, int dtype, int32_t d, int64_t n, uint8_t* out,
                                    int64_t row_offset, int32_t ld, int64_t rs, int64_t ws, float* inv_scale,
                                    const int32_t* tok_in, const int32_t* trace_in, const int32_t* prompt_in,
                                    int32_t* tok_out, int32_t* trace_out, int32_t* prompt_out, hipStream_t stream)
{
    const int ni = (ld + (FMT == kKeyFp8 ? 1024 : 512) - 1) / (FMT == kKeyFp8 ? 1024 : 512);  // 8 rows per workgroup
    const bool vec = ((int64_t)d * (dtype == 0 ? 4 : 2)) % 16 == 0;
    // NI iterations hold R rows, so that two workgroups fit a compute unit (one
    // loads while the other rounds): past 64 to 80 registers of raw values per
    // thread, four rows to a workgroup.  20,000 rows, us, 8 against 4 rows:
    // f32 to fp8 5,120 / 8,192 wide 145 / 231 against 130 / 172; bf16 to fp8
    // 69 / 149 against 85 / 118; f32 to bf16 127 / 220 against 143 / 216; bf16
    // to bf16 8,192 wide 143 against 168.
    auto go = [&](auto kernel, int R) {
        const int64_t groups = (row_offset + n - 1) / R - row_offset / R + 1;
        hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(kBulkThreads), 0, stream, raw, d, n, out, row_offset,
                           ld, rs, ws, inv_scale, tok_in, trace_in, prompt_in, tok_out, trace_out, prompt_out);
    };
    auto by_width = [&](auto f32, auto v) {
        constexpr bool F = decltype(f32)::value, V = decltype(v)::value;
        if constexpr (FMT == kKeyFp8) {
            if (V && ni <= 2) go(store_rows_kernel<FMT, F, V, V ? 2 : 4, 8>, 8);
            else if (ni <= 4) go(store_rows_kernel<FMT, F, V, 4, 8>, 8);
            else if (V && !F && ni <= 5) go(store_rows_kernel<FMT, F, V, V && !F ? 5 : 4, V && !F ? 8 : 4>, 8);
            else if (V && ni <= 6) go(store_rows_kernel<FMT, F, V, V ? 3 : 4, 4>, 4);
            else go(store_rows_kernel<FMT, F, V, 4, 4>, 4);
        } else {
            if (V && ni <= 4) go(store_rows_kernel<FMT, F, V, V ? 4 : 8, 8>, 8);
            else if (ni <= 8) go(store_rows_kernel<FMT, F, V, 8, 8>, 8);
            else if (V && ni <= 10) go(store_rows_kernel<FMT, F, V, V ? 10 : 8, V ? 8 : 4>, 8);
            else if (V && !F) go(store_rows_kernel<FMT, F, V, V && !F ? 16 : 8, V && !F ? 8 : 4>, 8);
            else go(store_rows_kernel<FMT, F, V, 8, 4>, 4);
        }
    };
    if (dtype == 0)
        vec ? by_width(std::true_type{}, std::true_type{}) : by_width(std::true_type{}, std::false_type{});
    else
        vec ? by_width(std::false_type{}, std::true_type{}) : by_width(std::false_type{}, std::false_type{});
    return hipGetLastError();
}

hipError_t launch_quantize_rows(const void* raw, int dtype, int32_t d, int64_t n_rows_in, int64_t n_rows_out,
                                uint8_t* out, int64_t row_offset, int32_t ld8, int64_t rs_bytes,
                                int64_t ws_bytes, float* inv_scale, const int32_t* tok_in,
                                const int32_t* trace_in, const int32_t* prompt_in, int32_t* tok_out,
                                int32_t* trace_out, int32_t* prompt_out, hipStream_t stream)
{
    if (n_rows_out <= 0)
        return hipSuccess;
    if (tok_out && rs_bytes > 0 && n_rows_in == n_rows_out && bulk_rows(n_rows_in, ld8))
        return launch_store_rows<kKeyFp8>(raw, dtype, d, n_rows_in, out, row_offset, ld8, rs_bytes, ws_bytes,
                                          inv_scale, tok_in, trace_in, prompt_in, tok_out, trace_out, prompt_out,
                                          stream);
    hipLaunchKernelGGL(quantize_rows_kernel, dim3((unsigned)n_rows_out), dim3(kRowThreads), 0, stream, raw, dtype, d,
                       n_rows_in, out, row_offset, ld8, rs_bytes, ws_bytes, inv_scale, tok_in, trace_in,
                       prompt_in, tok_out, trace_out, prompt_out);
    return hipGetLastError();
}

hipError_t launch_normalize_rows(const void* raw, int dtype, int32_t d, int64_t n_rows_in,
                                 int64_t n_rows_out, uint16_t* out, int64_t row_offset, int32_t ld,
                                 int layout, int64_t rs, int64_t ws, const int32_t* tok_in,
                                 const int32_t* trace_in, const int32_t* prompt_in, int32_t* tok_out,
                                 int32_t* trace_out, int32_t* prompt_out, hipStream_t stream)
{
    if (n_rows_out <= 0)
        return hipSuccess;
    if (tok_out && layout == kLayoutTiled && n_rows_in == n_rows_out && bulk_rows(n_rows_in, ld))
        return launch_store_rows<kKeyBf16>(raw, dtype, d, n_rows_in, (uint8_t*)out, row_offset, ld, 2 * rs, 2 * ws,
                                           nullptr, tok_in, trace_in, prompt_in, tok_out, trace_out, prompt_out,
                                           stream);
    hipLaunchKernelGGL(normalize_rows_kernel, dim3((unsigned)n_rows_out), dim3(kRowThreads), 0, stream, raw,
                       dtype, d, n_rows_in, out, row_offset, ld, layout, rs, ws, tok_in, trace_in,
                       prompt_in, tok_out, trace_out, prompt_out);
    return hipGetLastError();
}

}  // namespace oil
