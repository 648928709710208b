// fp32 products on the bf16 matrix cores (internal).
//
// A float is split into three bf16 numbers, x = x0 + x1 + x2: x0 is x rounded to bf16, x1 the rounded remainder, x2 the
// remainder of that.  Each step leaves at most half a unit of the 8-bit significand, so |x1| <= 2^-8 |x|, |x2| <= 2^-16 |x|
// and three of them hold all 24 bits of x.  A product of two such numbers is the sum of nine bf16 products, each exact in
// the fp32 accumulator's arithmetic; the six with i + j <= 2 are taken, the three dropped ones add up to at most
// 2^-23 (1 + 2^-9) of the product by these bounds; measured on random operands 2^-24.2 at most and 2^-28 on average, less than the
// rounding of one fp32 multiplication (2^-24, 2^-25.5).  (The decomposition and the six-product form are the known "three bf16 terms" emulation of single
// precision.)
//
// Why: v_mfma_f32_16x16x4_f32 keeps the vector ALU of its SIMD idle, v_mfma_f32_16x16x32_bf16 does not, and six of the latter
// do the work of eight of the former.  Measured on this chip, per SIMD: 14.5 ns against 8.3 ns an instruction (116 against
// 50 ns for a 16x16x32 product), a vector instruction adds 3 ns to the first and nothing (up to two per MFMA) to the second.
// Accuracy, against float64 on random data: relative error 1.6e-7 at K = 160 (fp32 MFMA 2.4e-7), 5.5e-7 at K = 1600
// (6.8e-7); with all nine products the same to two digits.
//
// Range: all of fp32's.  bf16 has fp32's exponents, so the small terms of a value below 1e-33 would be subnormal or lost.  Therefore
// the terms are those of 2^24 x: every fp32 value, subnormal ones included, is a multiple of 2^-149, its terms are multiples of 2^-125
// and none of them is subnormal.  A sum of products then carries 2^48, which comes off at the end; powers of two commute with every
// rounding, so ordinary results are the same bits as without them.  At the upper end an operand of 2^103 (1e31) or more, a result
// above 2^79 (6e23), an infinity or a NaN makes the scaled sum infinite or NaN (nothing added to such a sum makes it finite
// again).  A wavefront that finds one among its sums computes its tiles again from the unscaled operands on the fp32 matrix
// cores (product32): slower, but such values belong to networks that have diverged.
#pragma once
#include "common.hpp"

namespace split {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int PLANES = 3;

// two floats -> packed bf16 (round to nearest even), and what is left of them
__device__ __forceinline__ unsigned take(float& a, float& b) {
    const bf16x2 h = __builtin_convertvector(floatx2{a, b}, bf16x2);
    const unsigned u = __builtin_bit_cast(unsigned, h);
    a -= __uint_as_float(u << 16);
    b -= __uint_as_float(u & 0xffff0000u);
    return u;
}

constexpr float SCALE = 0x1p24f, UNSCALE = 0x1p-48f;
__device__ __forceinline__ float4 scaled(float4 v) { return make_float4(v.x * SCALE, v.y * SCALE, v.z * SCALE, v.w * SCALE); }

// Sums that are infinite or NaN: `spoil` gathers them (0 or NaN; a group of four large ones may overflow as well, at no harm),
// `spoiled` says whether any lane of the wavefront has one.
__device__ __forceinline__ float spoil(const floatx4& sum, float so_far) { return fmaf((sum[0] + sum[1]) + (sum[2] + sum[3]), 0.f, so_far); }
__device__ __forceinline__ bool spoiled(float gathered) { return __builtin_expect(__any(gathered != 0.f) != 0, 0); }

// acc += a . b on the fp32 matrix cores; a[j], b[j]: the lane's value at the same reduction index.  All lanes take part.
template <int N>
__device__ __forceinline__ floatx4 product32(const float (&a)[N], const float (&b)[N], floatx4 acc) {
#pragma unroll
    for (int j = 0; j < N; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc, 0, 0, 0);
    return acc;
}

// four consecutive values (scaled) -> their three planes, 8 bytes each
__device__ __forceinline__ void split4(float4 v, uint2 (&p)[PLANES]) {
#pragma unroll
    for (int i = 0; i < PLANES; ++i) p[i] = make_uint2(take(v.x, v.y), take(v.z, v.w));
}

// acc[.] += a . b over 32 reduction indices; a[plane], b[plane]: a lane's 8 values (k = 8 (lane / 16) ..)
__device__ __forceinline__ floatx4 mfma(const uint4& a, const uint4& b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The six products for TA x TB tiles, small ones first, each over all tiles before the next (independent accumulators
// follow each other).  sum[i][j] is 16x16: rows from a, columns from b.  The five small products (2^-8 and less of the leading one) have
// an accumulator of their own: what a matrix-core instruction rounds, it rounds to the size of its accumulator, so the leading sum
// is then rounded once per 32 reduction indices and not six times.
template <int TA, int TB>
__device__ __forceinline__ void product(const uint4 (&a)[TA][PLANES], const uint4 (&b)[TB][PLANES], floatx4 (&sum)[TA][TB], floatx4 (&small)[TA][TB]) {
    constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j) {
                floatx4& to = p < 5 ? small[i][j] : sum[i][j];
                to = mfma(a[i][PA[p]], b[j][PB[p]], to);
            }
}

// Transposing LDS read: the 16 lanes of a quarter wavefront name four rows of 16 two-byte elements (lane j: row j / 4,
// elements 4 (j mod 4) ..), lane j receives element j of each row.  Two of them give a lane eight consecutive reduction
// indices of its row or column out of a tile that is stored with the reduction index outermost.
typedef short shortx4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 read_tr(const char* lds) {
    typedef __attribute__((address_space(3))) shortx4 lds_t;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t*)lds));
}

// One matrix-core operand of (scaled) fp32 values.  32 reduction channels: the three planes, a lane's eight channels each.
// 16 reduction channels (C = 16): an instruction's 32 indices take two planes of them, a lane's four channels each, and
// three instructions instead of six do the six products: (y2, y0) . (x0, x2), (y1, y0) . (x0, x1), (y0, y1) . (x0, x1).
// A pixel operand is fetched as the two register quads it is used as, x0 twice: put together by moves, it takes ten more vector
// instructions, and as these wait for the fetch they follow, the fetch of the next operand no longer overlaps the products of the
// present one.
template <int C> struct Filt { uint4 v[3]; };
template <int C> struct Pix { uint4 v[C == 16 ? 2 : 3]; };

template <int C> __device__ __forceinline__ Filt<C> filter_operand(const float4 (&r)[C == 16 ? 1 : 2]) {
    Filt<C> f;
    uint2 lo[PLANES];
    split4(r[0], lo);
    if constexpr (C == 16) {
        f.v[0] = make_uint4(lo[2].x, lo[2].y, lo[0].x, lo[0].y);
        f.v[1] = make_uint4(lo[1].x, lo[1].y, lo[0].x, lo[0].y);
        f.v[2] = make_uint4(lo[0].x, lo[0].y, lo[1].x, lo[1].y);
    } else {
        uint2 hi[PLANES];
        split4(r[1], hi);
#pragma unroll
        for (int p = 0; p < PLANES; ++p) f.v[p] = make_uint4(lo[p].x, lo[p].y, hi[p].x, hi[p].y);
    }
    return f;
}

// at, again: the same address; C = 16 fetches x0 through both, where the compiler does not know that it is the same.  (The first layer of the
// AlexNet-style networks gives one address: its loop has the time for the moves and not for the reads, 1 to 2 % of a step.)
template <int C, int PLANE> __device__ __forceinline__ Pix<C> pixel_operand(const char* at, const char* again) {
    Pix<C> x;
    if constexpr (C == 16) {
        const uint2 a = *reinterpret_cast<const uint2*>(at), x2 = *reinterpret_cast<const uint2*>(at + 2 * PLANE),
                    b = *reinterpret_cast<const uint2*>(again), x1 = *reinterpret_cast<const uint2*>(again + PLANE);
        x.v[0] = make_uint4(a.x, a.y, x2.x, x2.y);
        x.v[1] = make_uint4(b.x, b.y, x1.x, x1.y);
    } else {
#pragma unroll
        for (int p = 0; p < PLANES; ++p) x.v[p] = *reinterpret_cast<const uint4*>(at + p * PLANE);
    }
    return x;
}

template <int C, int PLANE> __device__ __forceinline__ Pix<C> pixel_operand(const char* at) { return pixel_operand<C, PLANE>(at, at); }

// the same for the transposing reads of the d-filter step: lane l16 of quarter q receives channel l16 of pixels 8 q ..
template <int PLANE> __device__ __forceinline__ void transposed_operand(uint4 (&x)[PLANES], const char* lo_at, const char* hi_at) {
#pragma unroll
    for (int p = 0; p < PLANES; ++p) {
        const uint2 lo = read_tr(lo_at + p * PLANE), hi = read_tr(hi_at + p * PLANE);
        x[p] = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
}

template <int C> constexpr int products() { return C == 16 ? 3 : 6; }
// product p of the sum, small ones first
template <int C> __device__ __forceinline__ floatx4 product(int p, const Filt<C>& f, const Pix<C>& x, floatx4 acc) {
    if constexpr (C == 16) {
        return mfma(f.v[p], x.v[p ? 1 : 0], acc);
    } else {
        constexpr int PF[6] = {0, 2, 1, 0, 1, 0}, PX[6] = {2, 0, 1, 1, 0, 0};
        return mfma(f.v[PF[p]], x.v[PX[p]], acc);
    }
}

// Buffer loads check their offset against the buffer's size and return zero beyond it: zero padding without a branch and
// without a select.  Offsets are unsigned bytes below 2^32; OUTSIDE lies beyond any buffer of less than 2^31 bytes, also after
// another such offset is added to it.
constexpr unsigned OUTSIDE = 0x80000000u;
typedef __amdgpu_buffer_rsrc_t Buffer;
__device__ __forceinline__ Buffer buffer(const void* p, unsigned bytes) {
    constexpr int RAW_DWORDS = 0x00027000;          // untyped 32-bit data, no swizzle
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, RAW_DWORDS);
}
__device__ __forceinline__ float4 load4(Buffer b, unsigned offset) {
    return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)offset, 0, 0));
}
__device__ __forceinline__ float2 load2(Buffer b, unsigned offset) {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(b, (int)offset, 0, 0));
}
__device__ __forceinline__ unsigned load1(Buffer b, unsigned offset) { return __builtin_amdgcn_raw_buffer_load_b32(b, (int)offset, 0, 0); }

}  // namespace split
