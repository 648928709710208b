// Filters of the 3x3 kernels (conv3x3.hpp) converted once per step: every operand of the matrix cores that a wavefront needs, as the three
// bf16 terms of split.hpp.  A workgroup then neither splits the filter (68 vector instructions an operand and wavefront: in the workgroups for
// small batches, which have no second wavefront on a SIMD to multiply meanwhile, more time than the products) nor gathers it with a stride, and
// needs no registers for the floats (of 122 to 130 a lane 8 to 26 less).  A round of pushes without / with it, us: 110 layers, batch 128, eight
// workers 16216 / 16093, batch 3 7836 / 7677; 50 layers, batch 128 7548 / 7361, two workers, batch 8 1224 / 1143; 20 layers, batch 8, four workers
// 716 / 678, batch 17, three 611 / 580.
#pragma once
#include "split.hpp"

// A filter [3][3][C][C]: the floats, and its operands or NULL (the kernel splits the floats itself: callers of single layers).
struct Filter3x3 {
    const float* w;
    const uint4* planes;
    Filter3x3(const float* w_, const uint4* planes_ = nullptr) : w(w_), planes(planes_) {}
};

// Operands of one filter and direction: [tap][32 reduction channels][16 result channels][quad][lane].  Of the three quads of 16 reduction channels, (x2, x0),
// (x1, x0) and (x0, x1), the second is the third with its halves exchanged and is not stored (every
// wavefront of a workgroup fetches all of such a filter; a round of pushes with three / two quads, us: 110 layers, batch 128 15382 / 15310, 56 layers, batch 2
// 932 / 929, 20 layers, batch 8 475 / 473).
constexpr int filter3x3_quads(int C) { return C == 16 ? 2 : 3; }
constexpr int filter3x3_operands(int C) { return 9 * (C / 16) * (C == 16 ? 1 : C / 32); }
constexpr size_t filter3x3_uint4s(int C) { return (size_t)filter3x3_operands(C) * filter3x3_quads(C) * 64; }

// `count` filters of C channels, one every `stride` floats from `first` on.
struct FilterRun { int64_t first; int count, stride; };

// The conversion has no launch of its own: the first kernel of a step carries it as workgroups behind its own (a launch more is 4 us of a small
// network's push, and 3 % of one whose step is not a graph).
struct FilterJob {
    static constexpr int THREADS = 256;
    const float* w;
    uint4* out;             // the runs (C = 16, 32, 64) one after the other; of each filter forward, then d-input (taps reversed, channels swapped)
    FilterRun run[3];
    int end[3];             // operands up to and with the run
    int own_blocks;         // of the carrier

    FilterJob(const float* w_, uint4* out_, const FilterRun (&runs)[3]) : w(w_), out(out_), own_blocks(0) {
        int n = 0;
        for (int i = 0; i < 3; ++i) {
            run[i] = runs[i];
            end[i] = n += runs[i].count * 2 * filter3x3_operands(16 << i);
        }
    }
    int blocks() const { return (end[2] + THREADS / 64 - 1) / (THREADS / 64); }
};

template <int C>
__device__ __forceinline__ void convert_filter(const float* __restrict__ w, uint4* __restrict__ out, const FilterRun& run, int at, int lane) {
    constexpr int PER = filter3x3_operands(C), TILES = C / 16, FV = C == 16 ? 1 : 2;
    const int ct = at % TILES, c32 = at / TILES % (PER / 9 / TILES), tap = at % PER / (PER / 9), which = at / PER;
    const float* f = w + run.first + (int64_t)(which / 2) * run.stride;
    const int rs = 16 * ct + (lane & 15), k0 = C == 16 ? 4 * (lane >> 4) : 32 * c32 + 8 * (lane >> 4);
    float4 v[FV];
#pragma unroll
    for (int e = 0; e < FV; ++e) {
        if (which % 2) {
            v[e] = *reinterpret_cast<const float4*>(f + ((8 - tap) * C + rs) * C + k0 + 4 * e);
        } else {
            const float* p = f + (tap * C + k0 + 4 * e) * C + rs;
            v[e] = make_float4(p[0], p[C], p[2 * C], p[3 * C]);
        }
        v[e] = split::scaled(v[e]);
    }
    const split::Filt<C> terms = split::filter_operand<C>(v);
#pragma unroll
    for (int p = 0; p < filter3x3_quads(C); ++p) out[((int64_t)at * filter3x3_quads(C) + p) * 64 + lane] = terms.v[C == 16 ? 2 * p : p];
}

// Workgroup `block` of the job, a wavefront an operand.
__device__ __forceinline__ void convert_filters(const FilterJob& j, int block) {
    const int at = __builtin_amdgcn_readfirstlane(block * (FilterJob::THREADS / 64) + (int)threadIdx.x / 64), lane = threadIdx.x & 63;
    uint4* out = j.out;
    if (at < j.end[0]) return convert_filter<16>(j.w, out, j.run[0], at, lane);
    out += (int64_t)j.end[0] * filter3x3_quads(16) * 64;
    if (at < j.end[1]) return convert_filter<32>(j.w, out, j.run[1], at - j.end[0], lane);
    out += (int64_t)(j.end[1] - j.end[0]) * filter3x3_quads(32) * 64;
    if (at < j.end[2]) convert_filter<64>(j.w, out, j.run[2], at - j.end[1], lane);
}
