// The end of a residual network's step, one image to a workgroup: last batch norm with shortcut and ReLU, average pooling, the fully connected
// layer, softmax cross-entropy, and the way back to the masked gradient in front of that ReLU with its sum records.  All of it depends on one
// image, but for the statistics that its input brings as records; the gradients of the layer's weights sum over the images and remain dsspk_fc_bwd's.
// Bound by latency: a chain of five dependent stages of at most 1 us each, which as four launches (dsspk_bn_fwd_gap, dsspk_fc_softmax_xent, dx of
// dsspk_fc_bwd, dsspk_gap_bwd_bn_reduce) took 23 us at batch 8 and 28 at 128, with the image read three times.  A push with those / with this, us: 20 layers,
// batch 8, one worker 348.7 / 337.1, four 106.8 / 104.1; 50 layers, batch 128, one worker 1538 / 1522, four 759 / 748; 8 layers, batch 13, three
// workers, launches, a round 400 / 374.
#include "conv3x3.hpp"
#include "head.hpp"

namespace {

constexpr int HEAD_THREADS = 256, HEAD_WAVES = 4, HEAD_C = 64, HEAD_SIDE = 8, HEAD_PX = HEAD_SIDE * HEAD_SIDE;
static_assert(HEAD_THREADS == bnm::THREADS && HEAD_MAX_PARTS * HEAD_C == 32 * HEAD_THREADS, "the records a thread merges");
constexpr int HEAD_V = HEAD_C / 4, HEAD_ROWS = HEAD_THREADS / HEAD_V, HEAD_PER = HEAD_PX / HEAD_ROWS;    // a thread: 4 channels of every HEAD_ROWS-th pixel

// Sum over the pixels of the workgroup's image, in all threads of the four channels; red: HEAD_WAVES * HEAD_C floats.
__device__ __forceinline__ float4 image_sum(float4 v, float* red) {
    const int tid = threadIdx.x, vc = tid % HEAD_V;
    v = make_float4(lanes_sum<16>(v.x), lanes_sum<16>(v.y), lanes_sum<16>(v.z), lanes_sum<16>(v.w));
    if ((tid & 63) < HEAD_V) *reinterpret_cast<float4*>(red + tid / 64 * HEAD_C + 4 * vc) = v;
    __syncthreads();
    float4 s = *reinterpret_cast<const float4*>(red + 4 * vc);
#pragma unroll
    for (int w = 1; w < HEAD_WAVES; ++w) {
        const float4 o = *reinterpret_cast<const float4*>(red + w * HEAD_C + 4 * vc);
        s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
    }
    return s;
}

__global__ __launch_bounds__(HEAD_THREADS) void head_kernel(const float* __restrict__ records, const float* __restrict__ x, const float* __restrict__ shortcut,
                                                            const float* __restrict__ gamma, const float* __restrict__ w, int parts, int half, HeadArgs a) {
    constexpr int C = HEAD_C;
    __shared__ __attribute__((aligned(16))) float W[HEAD_C * HEAD_MAX_CLASSES];
    __shared__ __attribute__((aligned(16))) float red[4][HEAD_WAVES * C], norm[2 * C], pool[C];
    __shared__ float Z[2][HEAD_MAX_CLASSES], dlog[HEAD_MAX_CLASSES];
    const int tid = threadIdx.x, lane = tid & 63, vc = tid % HEAD_V, row = tid / HEAD_V, classes = a.classes;
    const long image_at = (long)blockIdx.x * HEAD_PX * C;
    const bnm::Records rec(records, C, parts);
    const float4 ga = *reinterpret_cast<const float4*>(gamma + 4 * vc), be = *reinterpret_cast<const float4*>(gamma + C + 4 * vc);
    const split::Buffer beside = split::buffer(shortcut + (half ? 2 : 1) * image_at, (half ? 8u : 4u) * HEAD_PX * C);
    float4 v[HEAD_PER], sc[HEAD_PER];
#pragma unroll
    for (int u = 0; u < HEAD_PER; ++u) {
        const int px = row + u * HEAD_ROWS;
        v[u] = *reinterpret_cast<const float4*>(x + image_at + px * C + 4 * vc);
        // a shortcut of twice the size and half the channels: every second pixel, zero beyond its channels
        const unsigned second = ((2 * (px / HEAD_SIDE) * 2 * HEAD_SIDE + 2 * (px % HEAD_SIDE)) * (C / 2) + 4 * vc) * 4u;
        sc[u] = split::load4(beside, !half ? (px * C + 4 * vc) * 4u : 4 * vc < C / 2 ? second : split::OUTSIDE);
    }
    constexpr int WV = C * HEAD_MAX_CLASSES / 4 / HEAD_THREADS;
    const split::Buffer weights = split::buffer(w, 4u * C * classes);
    float4 wv[WV];
#pragma unroll
    for (int u = 0; u < WV; ++u) wv[u] = split::load4(weights, 16u * (tid + u * HEAD_THREADS));
    const int y = a.label[blockIdx.x];
    const float bias = tid < classes ? w[C * classes + tid] : 0.f;

    // (merged as dsspk_bn_fwd_gap does, to the same bits)
    bnm::BnLayout L = {};
    L.G = parts;
    L.rows_per_block = a.rows_per_record;
    bnm::bn_merge_stats(rec, (long)parts * a.rows_per_record, C, a.eps, red[0], norm, L);
    if (blockIdx.x == 0 && tid < 2 * C) a.stats[tid] = norm[tid];
#pragma unroll
    for (int u = 0; u < WV; ++u)
        if (4 * (tid + u * HEAD_THREADS) < C * classes) *reinterpret_cast<float4*>(W + 4 * (tid + u * HEAD_THREADS)) = wv[u];
    const float4 mu = *reinterpret_cast<const float4*>(norm + 4 * vc), is = *reinterpret_cast<const float4*>(norm + C + 4 * vc);
    float4 hat[HEAD_PER], out[HEAD_PER], sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < HEAD_PER; ++u) {
        hat[u] = make_float4((v[u].x - mu.x) * is.x, (v[u].y - mu.y) * is.y, (v[u].z - mu.z) * is.z, (v[u].w - mu.w) * is.w);
        out[u].x = fmaxf(fmaf(hat[u].x, ga.x, be.x) + sc[u].x, 0.f);
        out[u].y = fmaxf(fmaf(hat[u].y, ga.y, be.y) + sc[u].y, 0.f);
        out[u].z = fmaxf(fmaf(hat[u].z, ga.z, be.z) + sc[u].z, 0.f);
        out[u].w = fmaxf(fmaf(hat[u].w, ga.w, be.w) + sc[u].w, 0.f);
        *reinterpret_cast<float4*>(a.out + image_at + (row + u * HEAD_ROWS) * C + 4 * vc) = out[u];
        sum.x += out[u].x; sum.y += out[u].y; sum.z += out[u].z; sum.w += out[u].w;
    }
    sum = image_sum(sum, red[0]);
    constexpr float INV = 1.f / HEAD_PX;
    sum = make_float4(sum.x * INV, sum.y * INV, sum.z * INV, sum.w * INV);
    if (tid < HEAD_V) {
        *reinterpret_cast<float4*>(pool + 4 * vc) = sum;
        *reinterpret_cast<float4*>(a.pooled + (long)blockIdx.x * C + 4 * vc) = sum;
    }
    __syncthreads();
    // logits: a thread half of a class's sum
    {
        const int c = tid % HEAD_MAX_CLASSES, k0 = tid / HEAD_MAX_CLASSES * (C / 2);
        float s = 0.f;
        if (c < classes)
#pragma unroll 8
            for (int k = k0; k < k0 + C / 2; ++k) s = fmaf(pool[k], W[k * classes + c], s);
        Z[tid / HEAD_MAX_CLASSES][c] = s + bias;            // (bias: zero in the second half)
    }
    __syncthreads();
    if (tid < 64) {
        float z[2], e[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) z[j] = lane + 64 * j < classes ? Z[0][lane + 64 * j] + Z[1][lane + 64 * j] : -INFINITY;
        float top = fmaxf(z[0], z[1]);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
        float se = 0.f;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            e[j] = lane + 64 * j < classes ? expf(z[j] - top) : 0.f;
            se += e[j];
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) se += __shfl_xor(se, o);
        const float inv = 1.0f / se;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int c = lane + 64 * j;
            if (c >= classes) continue;
            const float d = (e[j] * inv - (c == y ? 1.f : 0.f)) * a.inv_n;
            dlog[c] = d;
            a.logits[(long)blockIdx.x * classes + c] = z[j];
            a.dlogits[(long)blockIdx.x * classes + c] = d;
            if (c == y) a.row_loss[blockIdx.x] = logf(se) + top - z[j];
        }
    }
    __syncthreads();
    // gradient of the pooled values: four threads a channel
    {
        const int k = tid / 4;
        float s = 0.f;
#pragma unroll 4
        for (int c = tid % 4; c < classes; c += 4) s = fmaf(dlog[c], W[k * classes + c], s);
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        if (tid % 4 == 0) pool[k] = s * INV;
    }
    __syncthreads();
    const float4 g = *reinterpret_cast<const float4*>(pool + 4 * vc);
    float4 sb = make_float4(0.f, 0.f, 0.f, 0.f), sg = sb;
#pragma unroll
    for (int u = 0; u < HEAD_PER; ++u) {
        const float4 d = make_float4(out[u].x > 0.f ? g.x : 0.f, out[u].y > 0.f ? g.y : 0.f, out[u].z > 0.f ? g.z : 0.f, out[u].w > 0.f ? g.w : 0.f);
        *reinterpret_cast<float4*>(a.dz + image_at + (row + u * HEAD_ROWS) * C + 4 * vc) = d;
        sb.x += d.x; sb.y += d.y; sb.z += d.z; sb.w += d.w;
        sg.x = fmaf(d.x, hat[u].x, sg.x); sg.y = fmaf(d.y, hat[u].y, sg.y); sg.z = fmaf(d.z, hat[u].z, sg.z); sg.w = fmaf(d.w, hat[u].w, sg.w);
    }
    sb = image_sum(sb, red[1]);
    sg = image_sum(sg, red[2]);
    if (tid < HEAD_V) {
        float4* to = reinterpret_cast<float4*>(a.records_out + ((long)blockIdx.x * C + 4 * vc) * 2);
        to[0] = make_float4(sb.x, sg.x, sb.y, sg.y);
        to[1] = make_float4(sb.z, sg.z, sb.w, sg.w);
    }
}

}  // namespace

int resnet_head(hipStream_t s, const float* x, const float* records, int parts, const float* gamma, const float* shortcut, bool half, const float* w, int N,
                const HeadArgs& a) {
    if (!x || !records || !gamma || !shortcut || !w || N < 1 || !resnet_head_takes(N, parts, a.classes)) return -1;
    if (a.records_out == records || a.dz == x || a.out == x) return -1;       // other workgroups still read them
    hipLaunchKernelGGL(head_kernel, dim3(N), dim3(HEAD_THREADS), 0, s, records, x, shortcut, gamma, w, parts, half ? 1 : 0, a);
    return DSSPK_LAUNCH_RC();
}
