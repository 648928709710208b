// Stride-1 convolutions of wide layers (channels multiples of 64, 3x3 or 5x5
// filters) with fp32 arithmetic on the bf16 matrix cores (split.hpp): forward, gradient w.r.t. the input (the same kernel on
// a transposed, reversed filter) and gradient w.r.t. the filter and bias.
#include <algorithm>

#include "jobs.hpp"
#include "mma.hpp"
#include "split.hpp"
#include "conv_split_layers.hpp"
#include "../../include/dssp_kernels.h"

namespace {

using split_filter::BF16_NAN;
using split_filter::Frag;
using split_filter::filter_frag;

constexpr int THREADS = 256;
constexpr size_t LDS_MAX = 160 * 1024;

// ---------------------------------------------------------------------------------------------
// the value again from its terms (16 bits each)
__device__ __forceinline__ float filter_value(unsigned t0, unsigned t1, unsigned t2) {
    if ((t0 & 0x7fffu) == BF16_NAN) return __uint_as_float(t1 << 16 | t2);
    return (__uint_as_float(t0 << 16) + (__uint_as_float(t1 << 16) + __uint_as_float(t2 << 16))) * (1.f / split::SCALE);
}

__global__ __launch_bounds__(THREADS) void filter_planes_kernel(Frag fwd, Frag bwd, long n) {
    const long i = (long)blockIdx.x * THREADS + threadIdx.x;
    if (i < n) {
        if (fwd.out) filter_frag(fwd, false, i);
    } else if (i < 2 * n) {
        if (bwd.out) filter_frag(bwd, true, i - n);
    }
}

// ---------------------------------------------------------------------------------------------
// forward / d-input.  A workgroup owns 64 result channels of up to 16 MT pixels: R whole output rows of one image, or G whole
// images.  The input tile with its halo goes to LDS once, already split into its three planes (every element is converted
// once, not once per tap), and serves all taps from there; a pixel's 32 channels of one plane are a 16-byte read per lane.
// The filter planes come straight from L2 into registers, two steps ahead.  The matrix-core tile is 16 channels (rows) x
// 16 pixels (columns), so a lane ends up with four consecutive channels of a pixel.  Four wavefronts share out the tile.  The
// largest tile, one workgroup to a compute unit, has eight, two to a SIMD, so that one multiplies while the other fetches: the
// other four do the same with the other half of the staged reduction channels (the traffic per product stays that of the large
// tile), and the two halves of a sum meet in LDS at the end.  The smaller tiles gain nothing from that: several of their
// workgroups share a compute unit, and with more than one stream eight wavefronts cost 4 % of a step at batch 37.
// Bound by the matrix cores: 64 -> 64 at 5x5 on 15x15, batch 128, is 2.46 M MFMAs = 17 us of them at 2.4 GHz (the chip runs
// them at 1.9).  Measured at batch 37 / 128: 18 / 31 us (largest tile with four wavefronts 12 % more).
// A wavefront fetches a pixel operand as 16-byte reads of 16 pixels side by side in the result, four parts of a pixel each.  LDS has 64
// banks and serves such a read in four steps of 16 lanes, 0-3, 12-15 and 20-27 in the first: pixels 0-3 and 12-15 of one part, 4-11 of the
// next (measured read by read).  No two of them share a bank if a pixel takes 32 bytes (mod 64) more than the one before, also where a tile
// goes on in the next row or image of the result: these are padded to the bank at which their first pixel would have followed.  Rows of
// 15 pixels, 5x5: 4 steps a read instead of 11 on average with 16 bytes behind a pixel and nothing behind a row.  The reads are not what
// bounds the kernels, so the gain is small: batch 128 30.4 -> 30.1 us, 512 105.6 -> 103.8; 3x3, 256 channels on 14x14, batch 64 82 -> 80.
struct LdsPitch { int px, row, image; };       // bytes
constexpr int BANKS = 256;                     // bytes

LdsPitch lds_pitch(int channels, bool padded, int R, int OW, int ks) {
    LdsPitch p;
    p.px = channels * 2 * split::PLANES + (padded ? 32 : 16);
    p.row = (OW + ks - 1) * p.px;
    if (padded) p.row += (unsigned)((1 - ks) * p.px) % BANKS;
    p.image = (R + ks - 1) * p.row;
    if (padded) p.image += (unsigned)((1 - ks) * p.row) % BANKS;
    return p;
}

struct Geom {
    int N, H, W, OH, OW, pad;      // input / output pixel grid of this pass
    int IC, OC;                    // reduction / result channels of this pass
    int R, G, bands;               // output rows per tile, images per tile (G > 1: whole images), tiles per image
    LdsPitch at;                   // forward / d-input: the tile in LDS
};

// MT pixel tiles per workgroup; four wavefronts: WP over the pixels, 4 / WP over the 4 channel tiles; HALVES such groups
template <int MT> struct Waves { static constexpr int WP = MT >= 4 ? 2 : 1, WC = 4 / WP, TP = MT / WP, TC = 4 / WC, HALVES = MT == 8 ? 2 : 1; };

constexpr int ICB = 64;            // reduction channels staged at a time

// One pixel's four result channels 16 ct + 4 q ..: bias, addend, ReLU.
__device__ __forceinline__ void finish_pixel(const floatx4& sum, int ct, long at, const float* __restrict__ bias, const float* __restrict__ add,
                                             float* __restrict__ dst, int relu) {
    if (at < 0) return;
    const int co = 16 * ct + 4 * ((threadIdx.x & 63) >> 4);
    const float4 b = bias ? *reinterpret_cast<const float4*>(bias + co) : make_float4(0.f, 0.f, 0.f, 0.f);
    float4 v = make_float4(sum[0] + b.x, sum[1] + b.y, sum[2] + b.z, sum[3] + b.w);
    if (add) {
        const float4 a = *reinterpret_cast<const float4*>(add + at + co);
        v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
    }
    if (relu) { v.x = fmaxf(v.x, 0.f); v.y = fmaxf(v.y, 0.f); v.z = fmaxf(v.z, 0.f); v.w = fmaxf(v.w, 0.f); }
    *reinterpret_cast<float4*>(dst + at + co) = v;
}

// Sums beyond the range of the scaled terms: a matrix-core tile (16 channels, this lane's pixel of image n, row h0, column c) from the
// operands in memory.  A step takes 32 channels of a tap, a lane the eight of its filter fragment.
template <int KS>
__device__ __forceinline__ floatx4 direct_sum(const float* __restrict__ src, const uint4* __restrict__ wf, const Geom& g, int ct, int n, int h0,
                                              int c, bool ok) {
    const int lane = threadIdx.x & 63, q = lane >> 4, tiles_c = g.OC / 16, steps_c = g.IC / 32;
    floatx4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int tap = 0; tap < KS * KS; ++tap) {
        const int h = h0 + tap / KS - g.pad, w = c + tap % KS - g.pad;
        const bool in = ok && (unsigned)h < (unsigned)g.H && (unsigned)w < (unsigned)g.W;
        const float* px = src + (((long)n * g.H + h) * g.W + w) * g.IC + 8 * q;
        for (int c32 = 0; c32 < steps_c; ++c32) {
            float a[8], b[8];
            unsigned u[split::PLANES][4];
#pragma unroll
            for (int k = 0; k < split::PLANES; ++k)
                *reinterpret_cast<uint4*>(u[k]) = wf[((tap * steps_c + c32) * tiles_c + ct) * (split::PLANES * 64) + k * 64 + lane];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                a[j] = filter_value(u[0][j / 2] >> 16 * (j & 1) & 0xffffu, u[1][j / 2] >> 16 * (j & 1) & 0xffffu, u[2][j / 2] >> 16 * (j & 1) & 0xffffu);
                b[j] = in ? px[32 * c32 + j] : 0.f;
            }
            sum = split::product32(a, b, sum);
        }
    }
    mma::drain();
    return sum;
}

template <int MT, int KS>
__global__ __launch_bounds__(256 * Waves<MT>::HALVES) __attribute__((amdgpu_waves_per_eu(2))) void conv_split_kernel(const float* __restrict__ src, const uint4* __restrict__ wf,
                                                             const float* __restrict__ bias, const float* __restrict__ add,
                                                             float* __restrict__ dst, Geom g, int relu) {
    using W = Waves<MT>;
    constexpr int PLANE = 2 * ICB, CS = ICB / 32 / W::HALVES;      // CS: steps per tap and block of channels
    constexpr int STEPS = KS * KS * CS, WD = MT == 2 ? 8 : MT == 4 ? 4 : 2, NT = THREADS * W::HALVES;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4, half = W::HALVES == 2 ? wave >> 2 : 0;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int n0 = tile / g.bands * g.G, r0 = tile % g.bands * g.R;
    const int TH = g.R + KS - 1, TW = g.OW + KS - 1;
    const int wp = (wave & 3) % W::WP, wc = (wave & 3) / W::WP;
    const int ct0 = blockIdx.y * 4 + wc * W::TC;           // first 16-channel tile of this wavefront

    // this lane's pixels: where their patch starts in LDS, and where they go
    int base[W::TP];
    long out[W::TP];
#pragma unroll
    for (int t = 0; t < W::TP; ++t) {
        int p = (wp * W::TP + t) * 16 + l16;
        asm("" : "+v"(p));              // or the compiler keeps what it worked out above for every tile in registers through the product loop
        const int per = g.R * g.OW, gi = p / per, rest = p - gi * per, r = rest / g.OW, c = rest - r * g.OW;
        const bool ok = gi < g.G && n0 + gi < g.N && r0 + r < g.OH;
        base[t] = (ok ? gi * g.at.image + r * g.at.row + c * g.at.px : 0) + 16 * q + 64 * half;
        out[t] = ok ? (((long)(n0 + gi) * g.OH + r0 + r) * g.OW + c) * g.OC : -1;
    }
    // Small products have accumulators of their own, except in the largest tile: its halves round each sum half as often, which keeps
    // it below the fp32 matrix cores' error (5x5: 3.9e-7 against 4.7e-7), and 32 more registers would leave no room on the SIMD for
    // another kernel's wavefronts.
    constexpr bool APART = W::HALVES == 1;
    floatx4 acc[W::TC][W::TP], small[APART ? W::TC : 1][APART ? W::TP : 1];
#pragma unroll
    for (int i = 0; i < W::TC; ++i)
#pragma unroll
        for (int t = 0; t < W::TP; ++t) {
            acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};
            if constexpr (APART) small[i][t] = acc[i][t];
        }

    const int tiles_c = g.OC / 16, steps_c = g.IC / 32;
    const split::Buffer images = split::buffer(src + (long)n0 * g.H * g.W * g.IC, 4u * (unsigned)(min(g.G, g.N - n0) * g.H * g.W * g.IC));
    for (int c0 = 0; c0 < g.IC; c0 += ICB) {
        if (c0) __syncthreads();
        // Filter planes are fetched WD steps before their use (they come from L2: one step, 0.3 us, does not cover that),
        // pixel operands one step.
        uint4 wv[WD][W::TC][split::PLANES];
        auto load_w = [&](int buf, int s) {
            s = s < STEPS ? s : STEPS - 1;
            const uint4* p = wf + ((s / CS * steps_c + c0 / 32 + half + s % CS) * tiles_c + ct0) * (split::PLANES * 64) + lane;
#pragma unroll
            for (int i = 0; i < W::TC; ++i)
#pragma unroll
                for (int k = 0; k < split::PLANES; ++k) wv[buf][i][k] = p[(i * split::PLANES + k) * 64];
        };
#pragma unroll
        for (int u = 0; u < WD; ++u) load_w(u, u);
        // LOADS 16-byte loads in flight per thread (one at a time, their latencies add up to half the kernel)
        constexpr int LOADS = 8;
        const int total = g.G * TH * TW * (ICB / 4);
        for (int i0 = tid; i0 < total; i0 += LOADS * NT) {
            float4 v[LOADS];
            int to[LOADS];
#pragma unroll
            for (int e = 0; e < LOADS; ++e) {
                const int idx = i0 + e * NT, px = idx / (ICB / 4), c4 = idx % (ICB / 4);
                const int gi = px / (TH * TW), rest = px - gi * (TH * TW), ty = rest / TW, tx = rest - ty * TW;
                const int h = r0 + ty - g.pad, w = tx - g.pad;
                to[e] = gi * g.at.image + ty * g.at.row + tx * g.at.px + 8 * c4;
                const bool in = idx < total && (unsigned)h < (unsigned)g.H && (unsigned)w < (unsigned)g.W;      // images past the last: beyond the buffer
                v[e] = split::load4(images, in ? 4u * (unsigned)(((gi * g.H + h) * g.W + w) * g.IC + c0 + 4 * c4) : split::OUTSIDE);
            }
#pragma unroll
            for (int e = 0; e < LOADS; ++e) {
                if (i0 + e * NT >= total) break;
                uint2 pl[split::PLANES];
                split::split4(split::scaled(v[e]), pl);
#pragma unroll
                for (int p = 0; p < split::PLANES; ++p)
                    *reinterpret_cast<uint2*>(lds + to[e] + p * PLANE) = pl[p];
            }
        }
        uint4 pv[2][W::TP][split::PLANES];
        auto load_p = [&](int buf, int s) {
            s = s < STEPS ? s : STEPS - 1;
            const int tap = s / CS, off = tap / KS * g.at.row + tap % KS * g.at.px + s % CS * 64;
#pragma unroll
            for (int t = 0; t < W::TP; ++t)
#pragma unroll
                for (int k = 0; k < split::PLANES; ++k) pv[buf][t][k] = *reinterpret_cast<const uint4*>(lds + base[t] + off + k * PLANE);
        };
        __syncthreads();
        load_p(0, 0);
        for (int s = 0; s < STEPS; s += WD) {
#pragma unroll
            for (int u = 0; u < WD; ++u) {
                if (s + u >= STEPS) break;
                load_p((u + 1) & 1, s + u + 1);
                __builtin_amdgcn_sched_barrier(0);      // or the compiler moves the reads down to their use, behind the products
                if constexpr (APART) split::product(wv[u], pv[u & 1], acc, small);
                else split::product(wv[u], pv[u & 1], acc, acc);
                __builtin_amdgcn_sched_barrier(0);
                load_w(u, s + u + WD);
            }
        }
    }

    if constexpr (APART) {
#pragma unroll
        for (int i = 0; i < W::TC; ++i)
#pragma unroll
            for (int t = 0; t < W::TP; ++t) acc[i][t] += small[i][t];
    }
    auto direct = [&](int ct, int t) {
        int p = (wp * W::TP + t) * 16 + l16;
        asm("" : "+v"(p));              // or the compiler keeps what it worked out above for every tile in registers through the product loop
        const int per = g.R * g.OW, gi = p / per, rest = p - gi * per, r = rest / g.OW, c = rest - r * g.OW;
        const bool ok = gi < g.G && n0 + gi < g.N && r0 + r < g.OH;
        finish_pixel(direct_sum<KS>(src, wf, g, ct, n0 + gi, r0 + r, c, ok), ct, ok ? (((long)(n0 + gi) * g.OH + r0 + r) * g.OW + c) * g.OC : -1, bias, add,
                     dst, relu);
    };
    float bad = 0.f;
    if constexpr (W::HALVES == 1) {
#pragma unroll
        for (int i = 0; i < W::TC; ++i)
#pragma unroll
            for (int t = 0; t < W::TP; ++t) bad = split::spoil(acc[i][t], bad);
        if (split::spoiled(bad)) {
#pragma unroll 1
            for (int i = 0; i < W::TC * W::TP; ++i) direct(ct0 + i / W::TP, i % W::TP);
            return;
        }
#pragma unroll
        for (int i = 0; i < W::TC; ++i)
#pragma unroll
            for (int t = 0; t < W::TP; ++t) finish_pixel(acc[i][t] * split::UNSCALE, ct0 + i, out[t], bias, add, dst, relu);
    } else {        // the other half's share of the channel tile this wavefront finishes, against its own share of the other one
        static_assert(W::HALVES == 1 || W::TC == 2, "a channel tile each");
        __syncthreads();
        floatx4* ex = reinterpret_cast<floatx4*>(lds);             // [wavefront][TP][64]
#pragma unroll
        for (int t = 0; t < W::TP; ++t) {
            const floatx4 u = acc[0][t], v = acc[W::TC - 1][t];
            ex[(wave * W::TP + t) * 64 + lane] = half ? u : v;
            acc[0][t] = half ? v : u;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < W::TP; ++t) {
            acc[0][t] += ex[((wave ^ 4) * W::TP + t) * 64 + lane];
            bad = split::spoil(acc[0][t], bad);
        }
        if (split::spoiled(bad)) {
#pragma unroll 1
            for (int t = 0; t < W::TP; ++t) direct(ct0 + half, t);
            return;
        }
#pragma unroll
        for (int t = 0; t < W::TP; ++t) finish_pixel(acc[0][t] * split::UNSCALE, ct0 + half, out[t], bias, add, dst, relu);
    }
}

// ---------------------------------------------------------------------------------------------
// The same with the largest tile for more tiles than compute units (walks_tiles): one workgroup of eight wavefronts to a compute
// unit.  Wavefronts 0 .. 3 and 4 .. 7 take the filter taps in turn; the two halves of a sum meet in LDS at the end of a tile.  A workgroup
// walks its tiles in blocks of 32 reduction channels; while one block is multiplied, the next one (of this tile or the next) is converted into
// the other LDS buffer between the products, and the one after that is on its way into registers: nothing is staged in front of the
// products but a workgroup's first block.  The halves' numbers of steps differ by one; the longer one takes its extra step in front of the
// barrier that both pass once a block.  Bound by the matrix cores at two thirds of the rate they hold on such operands alone.  5x5, 64 -> 64
// on 15x15, one workgroup to a tile / this, us: batch 160 54.4 / 49.4, 256 56.0 / 53.8, 257 80.3 / 70.8, 512 109.7 / 101.8.
constexpr int LTHREADS = 512, LARGE_LOADS = 4;
constexpr int LARGE_HALO = LARGE_LOADS * LTHREADS / 8;         // pixels of a tile with its halo at most

template <int KS>
__global__ __launch_bounds__(LTHREADS) __attribute__((amdgpu_waves_per_eu(2))) void conv_split_large_kernel(const float* __restrict__ src, const uint4* __restrict__ wf,
                                                             const float* __restrict__ bias, const float* __restrict__ add,
                                                             float* __restrict__ dst, Geom g, int relu, int blocks, int per_group, int buffer_bytes) {
    constexpr int TAPS = KS * KS, TP = 4, TC = 2, PLANE = 64;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4, half = wave >> 2, wp = wave & 1, wc = wave >> 1 & 1;
    const int TH = g.R + KS - 1, TW = g.OW + KS - 1, per = g.R * g.OW;
    const int ct0 = blockIdx.y * 4 + wc * TC;              // first 16-channel tile of this wavefront
    const int tile0 = xcd_tile(blockIdx.x, gridDim.x) * per_group, tile1 = min(blocks, tile0 + per_group);
    const int tiles_c = g.OC / 16, steps_c = g.IC / 32;

    // where this lane's pixels' patches start in LDS (a pixel beyond the tile, the image or the batch takes what is there: not stored)
    int base[TP];
#pragma unroll
    for (int t = 0; t < TP; ++t) {
        const int p = (wp * TP + t) * 16 + l16, gi = p / per, rest = p - gi * per, r = rest / g.OW, c = rest - r * g.OW;
        base[t] = (gi < g.G ? gi * g.at.image + r * g.at.row + c * g.at.px : 0) + 16 * q;
    }
    floatx4 acc[TC][TP];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int t = 0; t < TP; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    };

    // The thread's staged elements.  Rows above or below a single image fall outside its buffer, as do images past the last.
    float4 rv[LARGE_LOADS];
    unsigned off[LARGE_LOADS];
    int put[LARGE_LOADS];                                  // where they go in LDS
#pragma unroll
    for (int e = 0; e < LARGE_LOADS; ++e) {
        const int idx = tid + e * LTHREADS, px = idx >> 3, c4 = idx & 7;
        const int gi = px / (TH * TW), rest = px - gi * (TH * TW), ty = rest / TW, tx = rest - ty * TW, h = ty - g.pad, w = tx - g.pad;
        const bool in = gi < g.G && (unsigned)w < (unsigned)g.W && (g.G == 1 || (unsigned)h < (unsigned)g.H);
        off[e] = in ? 4u * (unsigned)(((gi * g.H + h) * g.W + w) * g.IC + 4 * c4) : split::OUTSIDE;
        put[e] = (gi < g.G ? gi * g.at.image + ty * g.at.row + tx * g.at.px : g.G * g.at.image) + 8 * c4;      // or behind the tile
    }
    const int staged = (g.G * TH * TW * 8 + 63) / 64;      // wavefronts' worth of elements
    int ft = tile0, fc = 0;                                // tile and channel block of the next fetch
    unsigned fo = 0;
    split::Buffer images;
    auto locate = [&]() {
        const int n0 = ft / g.bands * g.G, r0 = ft % g.bands * g.R;
        images = ft < tile1 ? split::buffer(src + (long)n0 * g.H * g.W * g.IC, 4u * (unsigned)(min(g.G, g.N - n0) * g.H * g.W * g.IC)) : split::buffer(src, 0);
        fo = 4u * (unsigned)(r0 * g.W * g.IC + 32 * fc);
    };
    auto advance = [&]() {
        if (++fc == steps_c) { fc = 0; ++ft; }
        locate();
    };
    auto fetch = [&](int e) { if (wave + 8 * e < staged) rv[e] = split::load4(images, off[e] + fo); };
    auto stage = [&](int e, char* buf) {
        if (wave + 8 * e >= staged) return;
        uint2 pl[split::PLANES];
        split::split4(split::scaled(rv[e]), pl);
#pragma unroll
        for (int p = 0; p < split::PLANES; ++p) *reinterpret_cast<uint2*>(buf + put[e] + p * PLANE) = pl[p];
    };

    // Filter planes are fetched two steps before their use, also over the end of a block; pixel operands one step.
    uint4 wv[2][TC][split::PLANES], pv[2][TP][split::PLANES];
    int wtap = half, wblk = 0, wpar = half;
    auto load_w = [&](int buf) {
        const uint4* p = wf + ((wtap * steps_c + wblk) * tiles_c + ct0) * (split::PLANES * 64) + lane;
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int k = 0; k < split::PLANES; ++k) wv[buf][i][k] = p[(i * split::PLANES + k) * 64];
        wtap += 2;
        if (wtap >= TAPS) {
            wpar ^= 1;
            wtap = wpar;
            if (++wblk == steps_c) wblk = 0;
        }
    };
    auto load_p = [&](int buf, int tap, const char* from) {
        const int o = tap / KS * g.at.row + tap % KS * g.at.px;
#pragma unroll
        for (int t = 0; t < TP; ++t)
#pragma unroll
            for (int k = 0; k < split::PLANES; ++k) pv[buf][t][k] = *reinterpret_cast<const uint4*>(from + base[t] + o + k * PLANE);
    };
    locate();
#pragma unroll
    for (int e = 0; e < LARGE_LOADS; ++e) fetch(e);
    load_w(0);
    load_w(1);
    advance();
#pragma unroll
    for (int e = 0; e < LARGE_LOADS; ++e) stage(e, lds);
#pragma unroll
    for (int e = 0; e < LARGE_LOADS; ++e) fetch(e);
    advance();
    clear();
    __syncthreads();
    load_p(0, half, lds);

    int parity = half, blk = 0, tile = tile0;              // this wavefront's first tap of the block
    char *cur = lds, *nxt = lds + buffer_bytes;
    while (tile < tile1) {
        const int n = (TAPS + 1 - parity) / 2;             // steps: the two halves of the workgroup differ by one
        // Step s works with pv[s mod 2], wv[s mod 2].  While it does, the next one's pixel operands arrive: of this block, or behind the block's
        // barrier the first ones of the next.
        auto multiply = [&](int buf) {
            __builtin_amdgcn_sched_barrier(0);
            split::product(wv[buf], pv[buf], acc, acc);
            __builtin_amdgcn_sched_barrier(0);
            load_w(buf);
        };
        auto step = [&](int buf, int s) {
            load_p(buf ^ 1, parity + 2 * (s + 1), cur);
            multiply(buf);
        };
        static_assert(TAPS / 2 >= LARGE_LOADS, "a staged element to a step, all of them in front of the last one");
        int s = 0;
#pragma unroll
        for (; s < LARGE_LOADS - 1; ++s) {                 // (the compiler is free to mix these with the products)
            stage(s, nxt);
            if (s == LARGE_LOADS - 2) stage(s + 1, nxt);
            step(s & 1, s);
            fetch(s);
            if (s == LARGE_LOADS - 2) fetch(s + 1);
        }
        advance();
        static_assert(LARGE_LOADS % 2 == 0, "the loop goes on with the odd step");
        for (; s + 2 < n; s += 2) { step(1, s); step(0, s + 1); }
        if (s + 1 < n) {        // one more in this half: its operands go where the other half has those of its last step
            step(1, s);
#pragma unroll
            for (int k = 0; k < split::PLANES; ++k) {
#pragma unroll
                for (int t = 0; t < TP; ++t) pv[1][t][k] = pv[0][t][k];
#pragma unroll
                for (int i = 0; i < TC; ++i) { const uint4 w = wv[0][i][k]; wv[0][i][k] = wv[1][i][k]; wv[1][i][k] = w; }
            }
        }
        __syncthreads();        // the same one for both halves: everything of the next block is staged, this one has been read
        load_p(0, parity ^ 1, nxt);
        multiply(1);
        parity ^= 1;
        if (++blk == steps_c) {
            // the other half's share of the channel tile this wavefront finishes, against its own share of the other one, through the
            // buffer that was just consumed
            const int n0 = tile / g.bands * g.G, r0 = tile % g.bands * g.R;
            floatx4* ex = reinterpret_cast<floatx4*>(cur);         // [wavefront][TP][64]
#pragma unroll
            for (int t = 0; t < TP; ++t) {
                const floatx4 u = acc[0][t], v = acc[1][t];
                ex[(wave * TP + t) * 64 + lane] = half ? u : v;
                acc[0][t] = half ? v : u;
            }
            __syncthreads();
            float bad = 0.f;
#pragma unroll
            for (int t = 0; t < TP; ++t) {
                acc[0][t] += ex[((wave ^ 4) * TP + t) * 64 + lane];
                bad = split::spoil(acc[0][t], bad);
            }
            __syncthreads();                                       // before the next block is staged there
            const int ct = ct0 + half;
            auto pixel = [&](int t, auto&& value) {
                int p = (wp * TP + t) * 16 + l16;
                asm("" : "+v"(p));      // or the compiler keeps what it works out here in registers through the product loop
                const int gi = p / per, rest = p - gi * per, r = rest / g.OW, c = rest - r * g.OW;
                const bool ok = gi < g.G && n0 + gi < g.N && r0 + r < g.OH;
                finish_pixel(value(n0 + gi, r0 + r, c, ok), ct, ok ? (((long)(n0 + gi) * g.OH + r0 + r) * g.OW + c) * g.OC : -1, bias, add, dst, relu);
            };
            if (split::spoiled(bad)) {
#pragma unroll 1
                for (int t = 0; t < TP; ++t) pixel(t, [&](int n, int h, int c, bool ok) { return direct_sum<KS>(src, wf, g, ct, n, h, c, ok); });
            } else {
#pragma unroll
                for (int t = 0; t < TP; ++t) pixel(t, [&](int, int, int, bool) { return acc[0][t] * split::UNSCALE; });
            }
            clear();
            blk = 0;
            ++tile;
        }
        char* t = cur; cur = nxt; nxt = t;
    }
}

// Tile of one launch: the number of 16-pixel tiles per workgroup, its rows and images.
struct Tiling { int mt, R, G, bands, blocks; LdsPitch at; size_t lds; };
constexpr int UNITS = 256;         // compute units, one workgroup of the largest tile each

bool tiling_for(Tiling& t, int mt, int N, int OH, int OW, int ks) {
    const int px = 16 * mt;
    if (OW > px) return false;
    t.mt = mt;
    t.R = px / OW < OH ? px / OW : OH;
    t.bands = ceil_div(OH, t.R);
    t.R = ceil_div(OH, t.bands);                          // even bands
    t.G = t.bands == 1 ? px / (OH * OW) : 1;
    if (t.G > N) t.G = N;
    t.at = lds_pitch(ICB, false, t.R, OW, ks);
    while (t.G > 1 && (size_t)t.G * t.at.image > LDS_MAX) --t.G;
    // Padded, but never at the price of a smaller tile, nor of the second workgroup of a compute unit (the two smaller tiles: registers admit two).
    // Without the latter / so, us: 5x5 on 29x29, batch 18 42.4 / 32.3, on 36x36, batch 10 41.2 / 31.4; 3x3 on 64x64, batch 5 22.7 / 17.2.
    const LdsPitch padded = lds_pitch(ICB, true, t.R, OW, ks);
    const size_t room = mt < 8 && (size_t)t.G * t.at.image <= LDS_MAX / 2 ? LDS_MAX / 2 : LDS_MAX;
    if ((size_t)t.G * padded.image <= room) t.at = padded;
    t.lds = (size_t)t.G * t.at.image;
    if (mt == 8 && t.lds < 32 * 1024) t.lds = 32 * 1024;  // exchange of sums: four matrix-core tiles of each of the eight wavefronts
    t.blocks = ceil_div(N, t.G) * t.bands;
    return t.lds <= LDS_MAX;
}

// The largest tile (fewest halo rows and filter reads per pixel) that still gives most compute units (192 of 256) a workgroup.  With 96 /
// 192 / 384 in its place, 5x5 on 15x15, us: batch 24 21.4 / 14.0 / 13.9, 48 27.0 / 21.9 / 19.2, 96 27.4 / 27.2 / 30.9, 128 33.7 / 32.6 /
// 35.3, 130 49.7 / 49.8 / 47.3, 192 50.2 / 50.2 / 50.8 (walked tiles from 129 images on); 3x3 on 7x7: batch 96 9.2 / 6.8 / 6.8, 256 13.8 /
// 9.8 / 9.7.
bool choose_tiling(Tiling& t, int N, int OH, int OW, int OC, int ks) {
    bool have = false;
    for (int mt = 8; mt >= 2; mt /= 2) {
        Tiling c;
        if (!tiling_for(c, mt, N, OH, OW, ks)) continue;
        if (!have || (long)t.blocks * (OC / 64) < 192) t = c;
        have = true;
    }
    return have;
}

template <int MT, int KS>
int launch_tile(hipStream_t s, const float* src, const uint4* wf, const float* bias, const float* add, float* dst, const Geom& g, int relu,
                const Tiling& t) {
    auto kern = conv_split_kernel<MT, KS>;
    static bool attr_set = false;       // raise the dynamic-LDS limit once per instantiation
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_MAX) != hipSuccess) return -1;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(t.blocks, g.OC / 64), dim3(THREADS * Waves<MT>::HALVES), t.lds, s, src, wf, bias, add, dst, g, relu);
    return DSSPK_LAUNCH_RC();
}

// Bytes of one of its two buffers: the tile and a pixel behind it, or the exchange (four matrix-core tiles of every wavefront).
int large_buffer(const Geom& g) { return std::max(g.G * g.at.image + g.at.px, 32 * 1024); }

template <int KS>
int launch_large(hipStream_t s, const float* src, const uint4* wf, const float* bias, const float* add, float* dst, const Geom& g, int relu,
                 const Tiling& t) {
    auto kern = conv_split_large_kernel<KS>;
    static bool attr_set = false;
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_MAX) != hipSuccess) return -1;
        attr_set = true;
    }
    // as many tiles to a workgroup as there would be rounds of workgroups
    const int per = ceil_div(t.blocks, std::max(1, UNITS / (g.OC / 64)));
    const int buffer = large_buffer(g);
    hipLaunchKernelGGL(kern, dim3(ceil_div(t.blocks, per), g.OC / 64), dim3(LTHREADS), 2 * buffer, s, src, wf, bias, add, dst, g, relu, t.blocks, per,
                       buffer);
    return DSSPK_LAUNCH_RC();
}

// More tiles of the largest kind than compute units: the kernel that stages a workgroup's next tile during the present one.  (One tile to a
// workgroup has nothing to overlap and its barriers cost 1 to 10 %: 5x5 at batch 128 31.2 / 31.6 us, 3x3 at batch 512 15.4 / 16.9.)
bool walks_tiles(const Tiling& t, const Geom& g, int ks) {
    return t.mt == 8 && (long)t.blocks * (g.OC / 64) > UNITS && (long)t.G * (t.R + ks - 1) * (g.OW + ks - 1) <= LARGE_HALO;
}

int launch_conv(hipStream_t s, const float* src, const uint4* wf, const float* bias, const float* add, float* dst, Geom g, int ks, int relu) {
    Tiling t;
    if (!choose_tiling(t, g.N, g.OH, g.OW, g.OC, ks)) return -1;
    g.R = t.R; g.G = t.G; g.bands = t.bands;
#define GO(MT) return ks == 5 ? launch_tile<MT, 5>(s, src, wf, bias, add, dst, g, relu, t) : launch_tile<MT, 3>(s, src, wf, bias, add, dst, g, relu, t)
    if (walks_tiles(t, g, ks)) {
        g.at = lds_pitch(32, true, g.R, g.OW, ks);         // (63 KB a buffer at most, over all tiles of LARGE_HALO pixels)
        return ks == 5 ? launch_large<5>(s, src, wf, bias, add, dst, g, relu, t) : launch_large<3>(s, src, wf, bias, add, dst, g, relu, t);
    }
    g.at = t.at;
    if (t.mt == 8) GO(8);
    if (t.mt == 4) GO(4);
    GO(2);
#undef GO
}

// ---------------------------------------------------------------------------------------------
// d-filter (and bias gradient), stage 1 of 2.  Workgroup (chunk, filter row kh and 32 input channels, 64 output channels)
// walks its chunk's pixel tiles (R whole output rows of one image, at most 64 pixels): the x rows that filter row kh meets
// and the dy rows go to LDS as planes, and dw[kh][kw][ci][co] += x[pixel + kw][ci] dy[pixel][co] is accumulated for all KS
// taps of the row with the pixels as reduction index, 32 to an MFMA.  Both operands need a lane's pixels side by side while
// LDS has the channels side by side: the transposing LDS reads turn them.  The next tile's loads are in flight while the
// matrix cores work.  Wavefront w: input channels 16 (w mod 2) .., output channels 32 (w / 2 mod 2) .., the first or second 32
// pixels of the tile (w / 4: two wavefronts to a SIMD, one multiplies while the other fetches); their sums meet in LDS at the end.
// Measured with the reduction at batch 37 / 128 / 512: 22.4 / 42.5 / 137 us (four wavefronts, reads behind the barrier: 1 / 2 / 13 us more).  With the
// workgroups of a chunk side by side on one XCD 8.8 instead of 46 MB are fetched at 128 and 35 instead of 183 at 512, and it takes 24.4 / 44.9 / 134.
// Output: partial[chunk][KS KS IC OC (+ OC bias sums, added up by the workgroups of filter row 0 and the first channels)].
constexpr int WG_PX = 64, WG_XPX = 96, CTHREADS = 512;
constexpr int XPITCH = 32 * 6 + 32, DPITCH = 64 * 6 + 32;      // 24 and 8 words (mod 32): four rows cover all banks once

template <int KS>
__global__ __launch_bounds__(CTHREADS) __attribute__((amdgpu_waves_per_eu(2))) void wgrad_split_kernel(const float* __restrict__ x, const float* __restrict__ dy,
                                                              float* __restrict__ partial, Geom g, int items_per_chunk, int with_bias) {
    constexpr int NX = (WG_XPX * 8 + CTHREADS - 1) / CTHREADS, ND = WG_PX * 16 / CTHREADS;      // 16-byte loads per thread and tile
    static_assert(WG_PX == 64 && WG_PX * 16 % CTHREADS == 0, "one run of 32 pixels per wavefront");
    constexpr int XBYTES = WG_XPX * XPITCH, BUF = XBYTES + WG_PX * DPITCH;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4, run = wave >> 2;
    const int ci_w = 16 * (wave & 1), co_w = 32 * (wave >> 1 & 1);         // this wavefront's first channels within the workgroup's
    const int kh = blockIdx.y % KS, ci0 = blockIdx.y / KS * 32, co0 = blockIdx.z * 64;
    const int TW = g.OW + KS - 1, P = g.R * g.OW;
    const int items = g.N * g.bands, i0 = blockIdx.x * items_per_chunk, i1 = min(items, i0 + items_per_chunk);
    const bool bias_role = with_bias && blockIdx.y == 0;

    // transposing reads: this lane names row 8 q + l16 / 4 (and the one four further) of its run of 32 pixels
    int xa[2], da[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int p = 32 * run + 8 * q + 4 * h + (l16 >> 2);
        const int r = p / g.OW, c = p - r * g.OW;
        xa[h] = (p < P ? (r * TW + c) * XPITCH : 0) + 8 * (l16 & 3) + 2 * ci_w;      // beyond P dy is zero
        da[h] = p * DPITCH + 8 * (l16 & 3) + 2 * co_w;
    }
    floatx4 acc[KS][2][1], small[KS][2][1];
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[k][i][0] = small[k][i][0] = floatx4{0.f, 0.f, 0.f, 0.f};
    float4 sb = make_float4(0.f, 0.f, 0.f, 0.f);

    // The thread's staged elements: NX of x, then ND of dy.  One tile is in LDS and worked on, the next one is in registers
    // and converted and written to the other LDS buffer element by element between the products (a vector instruction beside
    // an MFMA costs nothing), and the registers it frees take the loads of the tile after that.
    constexpr int NE = NX + ND;
    float4 rv[NE];
    unsigned off[NE];              // byte offset from the tile's first row; rows above or below the image fall outside its buffer
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const bool is_x = e < NX;
        const int idx = tid + (is_x ? e : e - NX) * CTHREADS, px = is_x ? idx >> 3 : idx >> 4, c4 = is_x ? idx & 7 : idx & 15;
        const int width = is_x ? TW : g.OW, r = px / width, c = px - r * width - (is_x ? g.pad : 0);
        const bool in = is_x ? px < WG_XPX && r < g.R && c >= 0 && c < g.W : px < P;
        off[e] = !in ? split::OUTSIDE : is_x ? 4u * (unsigned)(((r + kh - g.pad) * g.W + c) * g.IC + ci0 + 4 * c4)
                                             : 4u * (unsigned)((r * g.OW + c) * g.OC + co0 + 4 * c4);
    }
    int fn = i0 / g.bands, fr = i0 % g.bands * g.R;            // tile of the next fetch: image, first row
    split::Buffer xb, db;
    auto image = [&]() {
        xb = split::buffer(x + (long)fn * g.H * g.W * g.IC, 4u * (unsigned)(g.H * g.W * g.IC));
        db = split::buffer(dy + (long)fn * g.OH * g.OW * g.OC, 4u * (unsigned)(g.OH * g.OW * g.OC));
    };
    auto fetch = [&](int e) {
        rv[e] = e < NX ? split::load4(xb, off[e] + 4u * (unsigned)(fr * g.W * g.IC)) : split::load4(db, off[e] + 4u * (unsigned)(fr * g.OW * g.OC));
    };
    int fetched = 1;                                           // tiles fetched so far
    auto advance = [&]() {                                     // past the chunk's end: zeros, which change no bias sum
        if (i0 + fetched < i1) {
            fr += g.R;
            if (fr >= g.bands * g.R) { fr = 0; ++fn; }
            image();
        } else {
            xb = split::buffer(x, 0); db = split::buffer(dy, 0);
        }
        ++fetched;
    };
    auto stage = [&](int e, char* buf) {
        const float4 v = rv[e];
        if (e >= NX) { sb.x += v.x; sb.y += v.y; sb.z += v.z; sb.w += v.w; }
        uint2 pl[split::PLANES];
        split::split4(split::scaled(v), pl);
        const int idx = tid + (e < NX ? e : e - NX) * CTHREADS;
        if (e < NX && idx >= WG_XPX * 8) return;
        char* to = e < NX ? buf + (idx >> 3) * XPITCH + 8 * (idx & 7) : buf + XBYTES + (idx >> 4) * DPITCH + 8 * (idx & 15);
#pragma unroll
        for (int p = 0; p < split::PLANES; ++p) *reinterpret_cast<uint2*>(to + p * (e < NX ? 64 : 128)) = pl[p];
    };
    uint4 dv[2][split::PLANES], dn[2][split::PLANES], xv[2][1][split::PLANES], xn[1][split::PLANES];
    auto load_d = [&](uint4 (&to)[2][split::PLANES], const char* buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i) split::transposed_operand<128>(to[i], buf + XBYTES + da[0] + 32 * i, buf + XBYTES + da[1] + 32 * i);
    };
    auto load_x = [&](uint4 (&to)[1][split::PLANES], int kw, const char* buf) { split::transposed_operand<64>(to[0], buf + xa[0] + kw * XPITCH, buf + xa[1] + kw * XPITCH); };
    if (i0 < i1) {
        image();
#pragma unroll
        for (int e = 0; e < NE; ++e) fetch(e);
        advance();
#pragma unroll
        for (int e = 0; e < NE; ++e) stage(e, lds);
#pragma unroll
        for (int e = 0; e < NE; ++e) fetch(e);
        advance();
        __syncthreads();
        load_d(dn, lds);
        load_x(xn, 0, lds);
    }
    for (int item = i0; item < i1; ++item) {
        const char* cur = lds + ((item - i0) & 1) * BUF;
        char* nxt = lds + ((item - i0 + 1) & 1) * BUF;
#pragma unroll
        for (int p = 0; p < split::PLANES; ++p) { dv[0][p] = dn[0][p]; dv[1][p] = dn[1][p]; xv[0][0][p] = xn[0][p]; }
#pragma unroll
        for (int kw = 0; kw < KS; ++kw) {
            // Operands are read one step ahead.  In the last step the next tile is complete and this one consumed (its last
            // operands are in registers): the barrier goes here, so that its wait and the next tile's first reads hide behind products.
            if (kw + 1 < KS) {
                load_x(xv[(kw + 1) & 1], kw + 1, cur);
            } else {
                __syncthreads();
                load_d(dn, nxt);
                load_x(xn, 0, nxt);
            }
            __builtin_amdgcn_sched_barrier(0);
            constexpr int SS = KS - 1;                         // steps that stage the next tile
            if (kw < SS) {
#pragma unroll
                for (int e = kw * NE / SS; e < (kw + 1) * NE / SS; ++e) stage(e, nxt);
            }
            split::product(dv, xv[kw & 1], acc[kw], small[kw]);
#pragma unroll
            for (int m = 0; m < 12; ++m) {                     // one MFMA, a few vector instructions, ...
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (kw < SS) {
#pragma unroll
                for (int e = kw * NE / SS; e < (kw + 1) * NE / SS; ++e) fetch(e);
            }
        }
        advance();
    }
    float bad = 0.f;
#pragma unroll
    for (int kw = 0; kw < KS; ++kw)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            acc[kw][i][0] += small[kw][i][0];
            bad = split::spoil(acc[kw][i][0], bad);
        }
    if (split::spoiled(bad)) {      // beyond the range of the scaled terms: this wavefront's sums from the operands in memory, four pixels a step
#pragma unroll
        for (int kw = 0; kw < KS; ++kw) acc[kw][0][0] = acc[kw][1][0] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int item = i0; item < i1; ++item) {
            const int n = item / g.bands, row0 = item % g.bands * g.R;
            for (int p = 32 * run + q; p < 32 * run + 32; p += 4) {
                const int r = p / g.OW, c = p - r * g.OW;
                const bool ok = p < P && row0 + r < g.OH;
                const float* dp = dy + (((long)n * g.OH + row0 + r) * g.OW + c) * g.OC + co0 + co_w + l16;
                const float d0[1] = {ok ? dp[0] : 0.f}, d1[1] = {ok ? dp[16] : 0.f};
#pragma unroll
                for (int kw = 0; kw < KS; ++kw) {
                    const int h = row0 + r + kh - g.pad, w = c + kw - g.pad;
                    const bool in = ok && (unsigned)h < (unsigned)g.H && (unsigned)w < (unsigned)g.W;
                    const float xs[1] = {in ? x[(((long)n * g.H + h) * g.W + w) * g.IC + ci0 + ci_w + l16] : 0.f};
                    acc[kw][0][0] = split::product32(d0, xs, acc[kw][0][0]);
                    acc[kw][1][0] = split::product32(d1, xs, acc[kw][1][0]);
                }
            }
        }
        mma::drain();
    } else {
#pragma unroll
        for (int kw = 0; kw < KS; ++kw) { acc[kw][0][0] *= split::UNSCALE; acc[kw][1][0] *= split::UNSCALE; }
    }
    const long E = (long)KS * KS * g.IC * g.OC;
    float* outp = partial + blockIdx.x * (E + (with_bias ? g.OC : 0));
    // the sums over the other run: this wavefront finishes its output channel tile `run` and gives the other one away
    static_assert(8 * KS * 1024 <= 2 * BUF, "room for the exchange");
    __syncthreads();
    floatx4* ex = reinterpret_cast<floatx4*>(lds);             // [wavefront][tap][64]
#pragma unroll
    for (int kw = 0; kw < KS; ++kw) ex[(wave * KS + kw) * 64 + lane] = run ? acc[kw][0][0] : acc[kw][1][0];
    __syncthreads();
#pragma unroll
    for (int kw = 0; kw < KS; ++kw) {
        const floatx4 own = run ? acc[kw][1][0] : acc[kw][0][0];
        *reinterpret_cast<floatx4*>(outp + ((long)(kh * KS + kw) * g.IC + ci0 + ci_w + l16) * g.OC + co0 + co_w + 16 * run + 4 * q) =
            own + ex[((wave ^ 4) * KS + kw) * 64 + lane];
    }
    if (bias_role) {                                           // lanes of one channel group, in order
        __syncthreads();
        float4* red = reinterpret_cast<float4*>(lds);
        red[tid] = sb;
        __syncthreads();
        if (tid < 16) {
            float4 s = red[tid];
            for (int j = 1; j < CTHREADS / 16; ++j) { const float4 v = red[tid + 16 * j]; s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w; }
            *reinterpret_cast<float4*>(outp + E + co0 + 4 * tid) = s;
        }
    }
}

template <int KS>
int launch_wgrad(hipStream_t s, dim3 grid, const float* x, const float* dy, float* partial, const Geom& g, int items_per_chunk, int with_bias) {
    constexpr int bytes = 2 * (WG_XPX * XPITCH + WG_PX * DPITCH);
    auto kern = wgrad_split_kernel<KS>;
    static bool attr_set = false;
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) return -1;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, grid, dim3(CTHREADS), bytes, s, x, dy, partial, g, items_per_chunk, with_bias);
    return DSSPK_LAUNCH_RC();
}

bool wgrad_rows(Geom& g, int ks) {
    if (g.OW > WG_PX || g.OW + ks - 1 > WG_XPX) return false;
    int R = WG_PX / g.OW;
    if (R > WG_XPX / (g.OW + ks - 1)) R = WG_XPX / (g.OW + ks - 1);
    if (R > g.OH) R = g.OH;
    g.bands = ceil_div(g.OH, R);
    g.R = ceil_div(g.OH, g.bands);
    g.G = 1;
    return true;
}

// Chunks: at most one workgroup per compute unit (its LDS allows no second one, so one more workgroup than that doubles the
// kernel's time); the partial results (chunks times the filter) stay small beside the activations.
int wgrad_items(const Geom& g, int ks) {
    const int roles = ks * (g.IC / 32) * (g.OC / 64);
    int chunks = 256 / roles;
    if (chunks < 1) chunks = 1;
    const int items = g.N * g.bands;
    if (chunks > items) chunks = items;
    return ceil_div(items, chunks);
}

bool shape_ok(int H, int W, int Cin, int Cout, int k, int pad) {
    return (k == 3 || k == 5) && Cin >= 64 && Cin % 64 == 0 && Cout >= 64 && Cout % 64 == 0 && pad >= 0 && pad < k && H >= 1 && W >= 1 &&
           H + 2 * pad >= k && W + 2 * pad >= k;
}

// Filter elements (and the bias behind them) are counted in int, by the reduction with a stride of as many more.
bool filter_ok(int Cin, int Cout, int k) { return (long)k * k * Cin * Cout + Cout <= 1L << 30; }

Geom forward_geom(int N, int H, int W, int Cin, int Cout, int k, int pad) {
    Geom g = {};
    g.N = N; g.H = H; g.W = W; g.OH = H + 2 * pad - k + 1; g.OW = W + 2 * pad - k + 1; g.pad = pad; g.IC = Cin; g.OC = Cout;
    return g;
}

Geom backward_geom(int N, int H, int W, int Cin, int Cout, int k, int pad) {
    const Geom f = forward_geom(N, H, W, Cin, Cout, k, pad);
    Geom g = {};
    g.N = N; g.H = f.OH; g.W = f.OW; g.OH = H; g.OW = W; g.pad = k - 1 - pad; g.IC = Cout; g.OC = Cin;
    return g;
}

}  // namespace

extern "C" int dsspk_conv_split_covers(int N, int H, int W, int Cin, int Cout, int k, int pad) {
    if (N < 1 || !shape_ok(H, W, Cin, Cout, k, pad)) return 0;
    Geom f = forward_geom(N, H, W, Cin, Cout, k, pad), b = backward_geom(N, H, W, Cin, Cout, k, pad);
    if (!filter_ok(Cin, Cout, k)) return 0;
    if ((long)H * W * Cin >= 1L << 29 || (long)f.OH * f.OW * Cout >= 1L << 29) return 0;
    if ((long)N * H * W >= 1L << 31 || (long)N * f.OH * f.OW >= 1L << 31) return 0;
    // byte offsets within a group of images stay below split::OUTSIDE
    auto fits = [&](const Geom& g) { Tiling t; return choose_tiling(t, N, g.OH, g.OW, g.OC, k) && (long)t.G * g.H * g.W * g.IC < 1L << 29; };
    return fits(f) && fits(b) && wgrad_rows(f, k);
}

extern "C" int dsspk_conv_split_resident(int N, int H, int W, int Cin, int Cout, int k, int pad) {
    if (!dsspk_conv_split_covers(N, H, W, Cin, Cout, k, pad)) return 0;
    const Geom g = forward_geom(N, H, W, Cin, Cout, k, pad);
    Tiling t;
    choose_tiling(t, N, g.OH, g.OW, Cout, k);
    return t.mt == 8 ? 1 : (int)std::min<size_t>(2, LDS_MAX / t.lds);
}

extern "C" size_t dsspk_conv_split_filter_bytes(int Cin, int Cout, int k) { return (size_t)k * k * Cin * Cout * 2 * split::PLANES; }

extern "C" int dsspk_conv_split_filters(void* stream, const float* w, void* planes_fwd, void* planes_bwd, int Cin, int Cout, int k) {
    if (!w || (!planes_fwd && !planes_bwd) || (k != 3 && k != 5) || Cin < 64 || Cin % 64 || Cout < 64 || Cout % 64 || !filter_ok(Cin, Cout, k))
        return -1;
    const Frag f{w, (uint4*)planes_fwd, k * k, Cin, Cout}, b{w, (uint4*)planes_bwd, k * k, Cin, Cout};
    const long n = (long)k * k * Cin * Cout / 8;
    hipLaunchKernelGGL(filter_planes_kernel, dim3(ceil_div(2 * n, THREADS)), dim3(THREADS), 0, (hipStream_t)stream, f, b, n);
    return DSSPK_LAUNCH_RC();
}

extern "C" int dsspk_conv_split_fwd(void* stream, const float* x, const void* planes_fwd, const float* bias, float* y, int N, int H, int W,
                                    int Cin, int Cout, int k, int pad, int relu) {
    if (!x || !planes_fwd || !y || !dsspk_conv_split_covers(N, H, W, Cin, Cout, k, pad)) return -1;
    return launch_conv((hipStream_t)stream, x, (const uint4*)planes_fwd, bias, nullptr, y, forward_geom(N, H, W, Cin, Cout, k, pad), k, relu);
}

extern "C" int dsspk_conv_split_bwd_data(void* stream, const float* dy, const void* planes_bwd, const float* add, float* dx, int N, int H,
                                         int W, int Cin, int Cout, int k, int pad) {
    if (!dy || !planes_bwd || !dx || !dsspk_conv_split_covers(N, H, W, Cin, Cout, k, pad)) return -1;
    return launch_conv((hipStream_t)stream, dy, (const uint4*)planes_bwd, nullptr, add, dx, backward_geom(N, H, W, Cin, Cout, k, pad), k, 0);
}

extern "C" size_t dsspk_conv_split_wgrad_scratch_floats(int N, int H, int W, int Cin, int Cout, int k, int pad) {
    if (!dsspk_conv_split_covers(N, H, W, Cin, Cout, k, pad)) return 0;
    Geom g = forward_geom(N, H, W, Cin, Cout, k, pad);
    wgrad_rows(g, k);
    return (size_t)ceil_div(g.N * g.bands, wgrad_items(g, k)) * ((size_t)k * k * Cin * Cout + Cout);
}

int conv_split_bwd_weight_parts(hipStream_t stream, const float* x, const float* dy, float* dw, int with_bias, float* scratch, int N, int H, int W,
                                int Cin, int Cout, int k, int pad, jobs::Partials* waiting) {
    if (!x || !dy || !dw || !scratch || !dsspk_conv_split_covers(N, H, W, Cin, Cout, k, pad)) return -1;
    Geom g = forward_geom(N, H, W, Cin, Cout, k, pad);
    wgrad_rows(g, k);
    const int per = wgrad_items(g, k), chunks = ceil_div(g.N * g.bands, per);
    const dim3 grid(chunks, k * (Cin / 32), Cout / 64);
    if (const int rc = k == 5 ? launch_wgrad<5>(stream, grid, x, dy, scratch, g, per, with_bias) : launch_wgrad<3>(stream, grid, x, dy, scratch, g, per, with_bias)) return rc;
    *waiting = {scratch, dw, k * k * Cin * Cout + (with_bias ? Cout : 0), chunks, false};
    return 0;
}

extern "C" int dsspk_conv_split_bwd_weight(void* stream, const float* x, const float* dy, float* dw, int with_bias, float* scratch, int N,
                                           int H, int W, int Cin, int Cout, int k, int pad) {
    jobs::Partials p;
    if (const int rc = conv_split_bwd_weight_parts((hipStream_t)stream, x, dy, dw, with_bias, scratch, N, H, W, Cin, Cout, k, pad, &p)) return rc;
    return dsspk_wgrad_reduce(stream, p.partial, p.dw, p.E, p.chunks);
}
