// The wide convolutions (k_conv_split.hip) and the first layer (k_conv_first.hip) of the AlexNet-style networks inside the library: conversion of the
// filters as a job that another kernel carries, and d-filter kernels whose partial sums wait for a reduction.
#pragma once
#include "jobs.hpp"
#include "split.hpp"

// (A named namespace: SplitFilterJob has these as members and goes from one source file to another.)
namespace split_filter {

// Filter planes in operand order: [step][16 result channels][plane][lane] of 16 bytes, step = (tap, 32 reduction channels),
// lane (l16, q) holding the reduction channels 8 q .. 8 q + 7 of result channel l16.  A wavefront then fetches an operand
// as one contiguous KiB.  Written once per step, read by every workgroup of the layer's convolutions.
// A value that the terms cannot hold (2^103 or more, infinite, NaN) has NaN as its leading term, which spoils every sum it enters, and
// its two halves in the place of the others, where the computation in fp32 finds it.
//   TR = false: result channel = output channel;  true (d-input): result = input channel, taps reversed
constexpr float WIDE = 0x1p103f;
constexpr unsigned BF16_NAN = 0x7fc0u;
struct Frag {
    const float* w;
    uint4* out;
    int taps, IC, OC;       // of the layer
};

__device__ __forceinline__ void filter_frag(const Frag& f, bool tr, long idx) {
    const int RC = tr ? f.OC : f.IC, RS = tr ? f.IC : f.OC;      // reduction / result channels
    const int lane = (int)(idx & 63);
    const long r = idx >> 6;
    const int tiles = RS / 16, tile = (int)(r % tiles), step = (int)(r / tiles);
    const int c32 = step % (RC / 32), tap = step / (RC / 32);
    const int rs = 16 * tile + (lane & 15), rc = 32 * c32 + 8 * (lane >> 4);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        v[j] = tr ? f.w[((long)(f.taps - 1 - tap) * f.IC + rs) * f.OC + rc + j] : f.w[((long)tap * f.IC + rc + j) * f.OC + rs];
    float t[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = v[j] * split::SCALE;
#pragma unroll
    for (int p = 0; p < split::PLANES; ++p) {
        unsigned u[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) u[j] = split::take(t[2 * j], t[2 * j + 1]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (fabsf(v[j]) < WIDE) continue;               // (not so for NaN)
            const unsigned bits = __float_as_uint(v[j]), part = p == 0 ? BF16_NAN : p == 1 ? bits >> 16 : bits & 0xffffu;
            u[j / 2] = j % 2 ? (u[j / 2] & 0xffffu) | part << 16 : (u[j / 2] & 0xffff0000u) | part;
        }
        f.out[(r * split::PLANES + p) * 64 + lane] = make_uint4(u[0], u[1], u[2], u[3]);
    }
}

}  // namespace split_filter

// A step's wide filters, forward and d-input: the first layer's kernel carries their conversion as workgroups behind its own, a launch of 4.8 us less for
// each layer.
struct SplitFilterJob {
    static constexpr int THREADS = 256, MOST = 4;
    split_filter::Frag frag[MOST] = {};
    int end[MOST] = {}, n = 0;         // workgroups up to and with a conversion

    void add(const float* w, void* fwd, void* bwd, int channels, int k) {
        for (void* out : {fwd, bwd}) {
            frag[n] = {w, (uint4*)out, k * k, channels, channels};
            end[n] = blocks() + ceil_div((long)k * k * channels * channels / 8, THREADS);
            ++n;
        }
    }
    int blocks() const { return n ? end[n - 1] : 0; }
};

__device__ __forceinline__ void convert_filters(const SplitFilterJob& j, int block) {
    int i = 0;
    while (i + 1 < j.n && block >= j.end[i]) ++i;
    const long at = (long)(block - (i ? j.end[i - 1] : 0)) * SplitFilterJob::THREADS + threadIdx.x;
    const split_filter::Frag f = j.frag[i];
    if (at < (long)f.taps * f.IC * f.OC / 8) split_filter::filter_frag(f, i % 2, at);
}

int conv_first_pool_fwd(hipStream_t s, const float* x, const float* w, const float* bias, float* a, float* pooled, uint8_t* arg, int N, SplitFilterJob job);
int conv_first_pool_bwd_weight_parts(hipStream_t s, const float* x, const float* dpooled, const float* pooled, const uint8_t* arg, float* dw, float* scratch,
                                     int N, jobs::Partials* waiting);
int conv_split_bwd_weight_parts(hipStream_t stream, const float* x, const float* dy, float* dw, int with_bias, float* scratch, int N, int H, int W,
                                int Cin, int Cout, int k, int pad, jobs::Partials* waiting);
