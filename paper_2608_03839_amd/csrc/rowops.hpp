// Row normalisation helpers shared by the key store and the recycled pool
// (internal only).  NT is the block size (a multiple of 64); one block
// normalises one row at a time.
#pragma once

#include "common.hpp"

namespace oil {

__device__ __forceinline__ double load_raw(const void* raw, int dtype, int64_t at)
{
    if (dtype == 0)
        return (double)((const float*)raw)[at];
    return (double)bf16_bits_to_float(((const uint16_t*)raw)[at]);
}

// Block-wide sum of one double per thread of an NT-thread block, fixed order
// (wave xor-tree, then the wave totals added left to right in wave order).
// red holds NT / 64 doubles.
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* red)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        v += __shfl_xor(v, o, kWave);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        red[wave] = v;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int w = 1; w < NT / 64; w++)
        t += red[w];
    __syncthreads();
    return t;
}

// Columns t, t + NT, ... of one raw row (d values at row * d) in thread t of
// an NT-thread block, NV per thread, every load in flight at once (clamped
// addresses; columns at or past d read 0).  A dead row (live false, the
// whole block alike) reads nothing and is all zeros.  bf16 and f32 values
// are exact in float.
template <int NT, int NV>
__device__ __forceinline__ void load_row(const void* raw, int dtype, int64_t row, int32_t d, bool live,
                                         float (&v)[NV])
{
    const int t = threadIdx.x;
#pragma unroll
    for (int i = 0; i < NV; i++)
        v[i] = 0.f;
    if (!live)
        return;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int32_t j = i * NT + t;
        v[i] = (float)load_raw(raw, dtype, row * d + (j < d ? j : d - 1));
    }
#pragma unroll
    for (int i = 0; i < NV; i++)
        if (i * NT + t >= d)
            v[i] = 0.f;
}

// Sum of squares of the values load_row left in one thread, in double, in
// column order.
template <int NV>
__device__ __forceinline__ double sum_squares(const float (&v)[NV])
{
    double ss = 0.0;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const double x = v[i];
        ss += x * x;
    }
    return ss;
}

// A row's norm, and its reciprocal as a pair of floats (inv + inv_lo is 1 / norm
// to about 2^-48).  v * inv in float lies within two float ulps of the exact
// quotient (one rounding of inv, one of the product), so wherever that product
// is further than that from a rounding boundary of the stored format, both
// round to the same stored value.  The few values closer than twice that,
// about one in 8,000, are settled by the product's residual (to about 2^-45
// of the quotient), and what that leaves open, like rows of extreme norm, by
// the division and rounding in double that define the result.
struct RowScale {
    double norm;
    float inv, inv_lo;
    bool fast;
};

__device__ __forceinline__ RowScale row_scale(double norm)
{
    RowScale s;
    s.norm = norm;
    s.fast = norm >= 0x1p-60 && norm <= 0x1p60;  // inv and the products of ordinary values stay normal
    const double full = s.fast ? 1.0 / norm : 0.0;
    s.inv = (float)full;
    s.inv_lo = (float)(full - (double)s.inv);
    return s;
}

// What v / norm exceeds the float product q = v * inv by, to about 2^-45 of it.
__device__ __forceinline__ float quotient_rest(float v, float q, const RowScale& s)
{
    return fmaf(v, s.inv, -q) + v * s.inv_lo;
}

// Whether the quotient q is too close to the middle of two bf16 values (or
// too small a number) for its float bits to decide the rounding.
__device__ __forceinline__ bool bf16_near(float q)
{
    const uint32_t u = __float_as_uint(q);
    return ((u - 0x7FFCu) & 0xFFFFu) <= 8u || (u << 1) - 1u < (54u << 24);
}

// The bf16 value that v / norm rounds to, for q = v * inv with bf16_near(q).
// divided: set where the last bits of s.norm decide.
__device__ __forceinline__ uint16_t bf16_settle(float v, float q, const RowScale& s, bool& divided)
{
    const uint32_t u = __float_as_uint(q);
    const float mid = __uint_as_float((u & 0xFFFF0000u) | 0x8000u);
    const float above = (q - mid) + quotient_rest(v, q, s);  // q - mid is a few ulps: exact
    if (!s.fast || (u << 1) - 1u < (54u << 24) || !(fabsf(above) > fabsf(q) * 0x1p-40f)) {
        divided = true;
        return double_to_bf16_rne((double)v / s.norm);
    }
    return (uint16_t)((u >> 16) + ((above > 0.f) != (q < 0.f) ? 1u : 0u));
}

__device__ __forceinline__ uint16_t unit_bf16(float v, const RowScale& s, bool& divided)
{
    const float q = v * s.inv;
    if (!s.fast || bf16_near(q))
        return bf16_settle(v, q, s, divided);
    return (uint16_t)((__float_as_uint(q) + 0x8000u) >> 16);
}

// The norm of the raw row that starts at element `at`, by one wave (all lanes,
// the same row), with the additions of normalize_row<NT>: the same bits.  Kernels
// whose lanes hold whole chunks of a row sum its squares in another order.  That
// norm is within 2^-46 of this one, which leaves every value as it is that the
// residual settles (it stays 2^-40 away from the middle); only for the values
// that are divided, none at all in ordinary rows, do they need this one.
template <int NT, bool F32>
__device__ __attribute__((noinline)) double column_order_norm(const void* __restrict__ raw, int64_t at, int32_t d)
{
    double sum = 0.0;
#pragma unroll 1
    for (int w = 0; w < NT / 64; w++) {
        double ss = 0.0;
#pragma unroll 1
        for (int32_t j = w * 64 + (int)(threadIdx.x & 63); j < d; j += NT) {
            const double x = load_raw(raw, F32 ? 0 : 1, at + j);
            ss += x * x;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1)
            ss += __shfl_xor(ss, o, kWave);
        sum += ss;
    }
    return sqrt(sum);
}

// Gives the lanes that need it that norm of their row: lane l of a wave has row
// l % R, which starts at element `at`.  Every lane of the wave takes part.
template <int NT, bool F32, int R>
__device__ __forceinline__ void column_order_norms(bool need, const void* __restrict__ raw, int64_t at, int32_t d,
                                                   double& norm)
{
    constexpr uint64_t kRow0 = R == 1 ? ~0ull : R == 4 ? 0x1111111111111111ull : 0x0101010101010101ull;
    static_assert(R == 1 || R == 4 || R == 8, "rows per wave");
    const uint64_t wanted = __ballot(need);
#pragma unroll 1
    for (int r = 0; r < R; r++) {
        if (!(wanted & (kRow0 << r)))
            continue;
        const double exact = column_order_norm<NT, F32>(raw, __shfl(at, r, kWave), d);
        if ((int)(threadIdx.x & (R - 1)) == r)
            norm = exact;
    }
}

// Eight columns c .. c + 7 of the raw row that starts at element `at` (d
// columns; those past it read as zeros), in 16-byte pieces: one of bf16 or two
// of f32 values.  VEC: every piece of a row is 16-byte aligned (base and row
// stride), so it lies inside the row or past it whole; else element loads.
template <bool F32, bool VEC>
__device__ __forceinline__ void load_chunk(const void* __restrict__ raw, int64_t at, int32_t c, int32_t d,
                                           u32x4 (&x)[F32 ? 2 : 1])
{
    constexpr int P = F32 ? 2 : 1;  // pieces
#pragma unroll
    for (int p = 0; p < P; p++) {
        const int32_t c0 = c + p * (8 / P);
        if constexpr (VEC) {
            x[p] = *(const u32x4*)((const char*)raw + (at + (c0 < d ? c0 : 0)) * (F32 ? 4 : 2));
            if (c0 >= d)
                x[p] = u32x4{0, 0, 0, 0};
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++) {
                if constexpr (F32) {
                    const uint32_t v = ((const uint32_t*)raw)[at + (c0 + e < d ? c0 + e : 0)];
                    x[p][e] = c0 + e < d ? v : 0u;
                } else {
                    const int32_t ca = c0 + 2 * e, cb = ca + 1;
                    const uint32_t lo = ((const uint16_t*)raw)[at + (ca < d ? ca : 0)];
                    const uint32_t hi = ((const uint16_t*)raw)[at + (cb < d ? cb : 0)];
                    x[p][e] = (ca < d ? lo : 0u) | (cb < d ? hi << 16 : 0u);
                }
            }
        }
    }
}

// Column e of a chunk.
template <bool F32>
__device__ __forceinline__ float chunk_value(const u32x4 (&x)[F32 ? 2 : 1], int e)
{
    if constexpr (F32)
        return __uint_as_float(x[e >> 2][e & 3]);
    else
        return __uint_as_float((e & 1) ? x[0][e >> 1] & 0xFFFF0000u : x[0][e >> 1] << 16);
}

// A chunk's eight bf16 values of the unit row, and whether some of them need
// settling (settle_chunk_bf16).
template <bool F32>
__device__ __forceinline__ u32x4 unit_chunk_bf16(const u32x4 (&x)[F32 ? 2 : 1], const RowScale& sc, bool& near)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    u32x4 w;
    near = !sc.fast;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const float q0 = chunk_value<F32>(x, e) * sc.inv, q1 = chunk_value<F32>(x, e + 1) * sc.inv;
        near |= bf16_near(q0) || bf16_near(q1);
        w[e >> 1] = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)q0, (__bf16)q1});
    }
    return w;
}

// The same with every value settled (zeros for a zero or NaN row).
template <bool F32>
__device__ __forceinline__ u32x4 settle_chunk_bf16(const u32x4 (&x)[F32 ? 2 : 1], const RowScale& sc, bool& divided)
{
    u32x4 w = {0, 0, 0, 0};
    if (!(sc.norm > 0.0))
        return w;
    for (int e = 0; e < 8; e++) {  // rolled: one copy of the division in double
        float v = 0.f;
#pragma unroll
        for (int f = 0; f < 8; f++)
            v = f == e ? chunk_value<F32>(x, f) : v;
        const uint32_t bits = (uint32_t)unit_bf16(v, sc, divided) << ((e & 1) * 16);
#pragma unroll
        for (int q = 0; q < 4; q++)
            w[q] |= q == (e >> 1) ? bits : 0u;
    }
    return w;
}

// normalize_row for ld <= NT * NV: the row is read once into registers.
template <int NT, int NV, class Dst>
__device__ __forceinline__ void normalize_row_regs(const void* raw, int dtype, int64_t row, int32_t d,
                                                   int32_t ld, bool live, double* red, Dst dst)
{
    const int t = threadIdx.x;
    float v[NV];
    load_row<NT, NV>(raw, dtype, row, d, live, v);
    const RowScale sc = row_scale(sqrt(block_sum<NT>(sum_squares(v), red)));
    bool divided;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int32_t j = i * NT + t;
        if (j < ld)
            dst(j, (j < d && sc.norm > 0.0) ? unit_bf16(v[i], sc, divided) : (uint16_t)0);
    }
}

// Normalise one raw row (d values at row * d) of an NT-thread block: the sum
// of squares in double (thread t takes columns t, t + NT, ... in order, then
// the fixed block tree), each value divided by the norm in double and rounded
// once to bf16; columns d .. ld - 1 (and every column of a zero or dead row)
// get zeros.  dst(j, bits) stores column j.  Rows of up to 8 NT columns are
// read once, every load in flight together; wider rows in batches of eight
// loads per thread, twice.  For a given NT the arithmetic, and so every
// stored bit, is the same either way.
template <int NT, class Dst>
__device__ __forceinline__ void normalize_row(const void* raw, int dtype, int64_t row, int32_t d, int32_t ld,
                                              bool live, double* red, Dst dst)
{
    if (ld <= NT * 4) {
        normalize_row_regs<NT, 4>(raw, dtype, row, d, ld, live, red, dst);
        return;
    }
    if (ld <= NT * 8) {
        normalize_row_regs<NT, 8>(raw, dtype, row, d, ld, live, red, dst);
        return;
    }
    constexpr int kU = 8;
    const int t = threadIdx.x;
    double ss = 0.0;
    if (live) {
        for (int32_t j0 = 0; j0 < d; j0 += NT * kU) {
            double v[kU];
#pragma unroll
            for (int i = 0; i < kU; i++) {
                const int32_t j = j0 + i * NT + t;
                v[i] = load_raw(raw, dtype, row * d + (j < d ? j : d - 1));
            }
#pragma unroll
            for (int i = 0; i < kU; i++)
                if (j0 + i * NT + t < d)
                    ss += v[i] * v[i];
        }
    }
    const double norm = sqrt(block_sum<NT>(ss, red));
    for (int32_t j0 = 0; j0 < ld; j0 += NT * kU) {
        double v[kU];
#pragma unroll
        for (int i = 0; i < kU; i++) {
            const int32_t j = j0 + i * NT + t;
            v[i] = live ? load_raw(raw, dtype, row * d + (j < d ? j : d - 1)) : 0.0;
        }
#pragma unroll
        for (int i = 0; i < kU; i++) {
            const int32_t j = j0 + i * NT + t;
            if (j < ld)
                dst(j, (live && j < d && norm > 0.0) ? double_to_bf16_rne(v[i] / norm) : (uint16_t)0);
        }
    }
}

}  // namespace oil
