// Batch-norm statistics records and their merge, shared by the batch-norm kernels and by the
// convolution kernels that normalise their input while loading it.
//
// A record is (mean, sum of squared deviations from that mean) of one channel over a slab of
// rows; slabs have `rows_per_block` rows (the last one possibly fewer).  Records come either from
// bn_stats_partial_kernel (row slabs) or from the epilogue of a convolution kernel (one record per
// workgroup tile).  Every consumer merges them itself in its prologue (or records_merge_kernel ahead of it), in a fixed order: the batch norm kernels and
// the network's last one as bn_merge_stats does, to the same bits; the 3x3 convolutions wavefront by wavefront (conv3x3.hpp).
#pragma once
#include "common.hpp"

namespace bnm {

constexpr int THREADS = 256;

struct BnLayout {
    int VC, RL;          // 16-byte columns per row, row lanes per workgroup
    long rows_per_block;
    int G;               // slabs = workgroups of the partial kernels
};

__host__ __device__ inline BnLayout bn_layout(long M, int C) {
    BnLayout L;
    L.VC = C / 4;
    L.RL = THREADS / L.VC;
    const long gmax = 32L * (THREADS / C);          // the merge takes at most 32 slab results per lane
    long rpb = (M + gmax - 1) / gmax;
    if (rpb < 64) rpb = 64;
    rpb = (rpb + L.RL - 1) / L.RL * L.RL;
    L.rows_per_block = rpb;
    L.G = (int)((M + rpb - 1) / rpb);
    return L;
}

// Sum `v` over the lanes that share channel thread mod C (C a power of two up to 64), as a tree that adds the farther half of them at each step: over the
// wavefronts, then within them.  red: THREADS floats; result in all threads.
__device__ __forceinline__ float reduce_sub(float v, float* red, int C) {
    static_assert(THREADS == 4 * 64, "four wavefronts");
    const int lane = threadIdx.x & 63;
    red[threadIdx.x] = v;
    __syncthreads();
    float out = (red[lane] + red[lane + 128]) + (red[lane + 64] + red[lane + 192]);
    for (int o = 32; o >= C; o >>= 1) out += __shfl_xor(out, o);
    __syncthreads();
    return out;
}

// The records of channel thread mod C that this thread merges (G <= 32 * (THREADS / C): at most 32), eight loads in flight at a time and none beyond the
// list's end but in its last eight.  Apart from their use, so that a kernel's own loads go out behind them and not behind their sums.  With 32 loads
// always, the rows of a kernel asked for behind the sums and sums by a tree with a barrier a step / so, a push, us: 20 layers, batch 8, one worker
// 337.6 / 327.6, four 103.9 / 101.1; 50 layers, batch 128, one worker 1521 / 1508.
struct Records {
    float2 v[32];
    __device__ __forceinline__ Records(const float* __restrict__ partial, int C, int G) {
        const int SUB = THREADS / C, c = threadIdx.x % C, sub = threadIdx.x / C;
#pragma unroll
        for (int u0 = 0; u0 < 32; u0 += 8) {
            if (u0 * SUB >= G) {
#pragma unroll
                for (int u = u0; u < u0 + 8; ++u) v[u] = make_float2(0.f, 0.f);
                continue;
            }
#pragma unroll
            for (int u = u0; u < u0 + 8; ++u) v[u] = *reinterpret_cast<const float2*>(partial + ((long)min(sub + u * SUB, G - 1) * C + c) * 2);
        }
    }
};

// Merge of the slab results by the whole workgroup (THREADS / C lanes per channel):
// mean = sum n_g mean_g / M, M2 = sum (M2_g + n_g (mean_g - mean)^2).
// On return sh[c] = mean, sh[C + c] = 1 / sqrt(M2 / M + eps) for every channel.
__device__ __forceinline__ void bn_merge_stats(const Records& r, long M, int C, float eps, float* red, float* sh, const BnLayout& L) {
    const int SUB = THREADS / C;
    const int c = threadIdx.x % C, sub = threadIdx.x / C;
    // rows of slab g: all but the last are equal; slabs past the end get weight 0
    const float rows = (float)L.rows_per_block, last = (float)(M - (L.G - 1) * L.rows_per_block);
    auto weight = [&](int u) {
        const int g = sub + u * SUB;
        return g < L.G - 1 ? rows : g == L.G - 1 ? last : 0.f;
    };
    float s = 0.f;
#pragma unroll
    for (int u0 = 0; u0 < 32; u0 += 8) {
        if (u0 * SUB >= L.G) continue;
#pragma unroll
        for (int u = u0; u < u0 + 8; ++u) s = fmaf(weight(u), r.v[u].x, s);
    }
    const float mean = reduce_sub(s, red, C) / (float)M;
    float m2 = 0.f;
#pragma unroll
    for (int u0 = 0; u0 < 32; u0 += 8) {
        if (u0 * SUB >= L.G) continue;
#pragma unroll
        for (int u = u0; u < u0 + 8; ++u) {
            const float d = r.v[u].x - mean, n = weight(u);
            m2 += n > 0.f ? r.v[u].y + n * d * d : 0.f;
        }
    }
    m2 = reduce_sub(m2, red, C);
    if (sub == 0) {
        sh[c] = mean;
        sh[C + c] = 1.0f / sqrtf(m2 / (float)M + eps);
    }
    __syncthreads();
}

}  // namespace bnm
