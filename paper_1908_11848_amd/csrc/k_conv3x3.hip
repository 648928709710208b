// The 3x3 kernels of conv3x3.hpp with four wavefronts to a workgroup behind the launchers of the raw layers, the small kernel that
// merges statistics records, and the d-filter kernels of their own.
#include "conv3x3.hpp"
#include "conv3x3_layers.hpp"
#include "../../include/dssp_kernels.h"

namespace {

constexpr int THREADS = 256;

// ---- gradient w.r.t. the filter by minimal filtering F(3x3, 2x2):
//      dw[tap][ci][co] = sum over pixels x[pixel + tap][ci] dy[pixel][co]; per 2x2 tile of dy and its 4x4 patch of x,
//      dw += A^T [ (B^T x B) .* (G dy G^T) ] A with B^T = [1 0 -1 0; 0 1 1 0; 0 -1 1 0; 0 -1 0 1],
//      G = [1 0; .5 .5; .5 -.5; 0 1], A^T = [1 1 1 0; 0 1 -1 0; 0 1 1 1].  The sum over tiles is taken in the
//      transformed domain by the matrix cores, M_xi[ci][co] += sum over tiles XT_xi[ci][tile] DT_xi[tile][co]
//      (16 products instead of 36 per tile), and A^T M A is applied once at the end.
// One run of 16 tiles: the lane (l16, q) transforms, as scalars, the patch (its input channel) and the dy tile (its
// output channel) of tile 4q + s for each of the four MFMA steps s.  at(tile) locates a tile once; x_at(o, r, c) and
// d_at(o, i, j) fetch the patch and dy elements from there.
template <class At, class XAt, class DAt>
__device__ __forceinline__ void dfilter_run(floatx4 (&M)[16], int q, At at, XAt x_at, DAt d_at) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const auto tile = at(4 * q + s);
        float XT[16], DT[16];
        {
            float t[4][4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float x[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) x[r] = x_at(tile, r, c);
                t[0][c] = x[0] - x[2]; t[1][c] = x[1] + x[2]; t[2][c] = x[2] - x[1]; t[3][c] = x[3] - x[1];
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                XT[4 * a] = t[a][0] - t[a][2]; XT[4 * a + 1] = t[a][1] + t[a][2];
                XT[4 * a + 2] = t[a][2] - t[a][1]; XT[4 * a + 3] = t[a][3] - t[a][1];
            }
        }
        {
            float u[4][2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float d0 = d_at(tile, 0, j), d1 = d_at(tile, 1, j);
                u[0][j] = d0; u[1][j] = 0.5f * (d0 + d1); u[2][j] = 0.5f * (d0 - d1); u[3][j] = d1;
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                DT[4 * a] = u[a][0]; DT[4 * a + 1] = 0.5f * (u[a][0] + u[a][1]);
                DT[4 * a + 2] = 0.5f * (u[a][0] - u[a][1]); DT[4 * a + 3] = u[a][1];
            }
        }
#pragma unroll
        for (int xi = 0; xi < 16; ++xi) M[xi] = __builtin_amdgcn_mfma_f32_16x16x4f32(XT[xi], DT[xi], M[xi], 0, 0, 0);
    }
}

// dw = A^T M A; call after mma::drain().
__device__ __forceinline__ void dfilter_finish(const floatx4 (&M)[16], floatx4 (&dw)[9]) {
    floatx4 S[3][4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        S[0][b] = M[b] + M[4 + b] + M[8 + b];
        S[1][b] = M[4 + b] - M[8 + b];
        S[2][b] = M[4 + b] + M[8 + b] + M[12 + b];
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        dw[3 * r] = S[r][0] + S[r][1] + S[r][2];
        dw[3 * r + 1] = S[r][1] - S[r][2];
        dw[3 * r + 2] = S[r][1] + S[r][2] + S[r][3];
    }
}

// Up to this many values every workgroup merges the records itself; a kernel of its own for that takes 4 us of a stream's time.  That serves
// callers of the layers one by one: a network's step runs these kernels at 33 to 96 images, and then the lists are longer.
constexpr int INLINE_RECORDS = 2048;
static_assert(inline_records<16, 4>() == INLINE_RECORDS / 16 && inline_records<64, 4>() == INLINE_RECORDS / 64, "what the kernels fetch");
constexpr bool records_inline(int parts, int C) { return (C == 16 || C == 32 || C == 64) && parts >= 1 && (long)parts * C <= INLINE_RECORDS; }

// Statistics records -> mean[C], invstd[C].  One workgroup per 4 channels, 64 lanes per channel, so a lane
// fetches at most 8 records (all in flight together) and the kernel is a few microseconds of latency on
// C/4 CUs; cheaper than letting every workgroup of the consumer repeat the merge.  The arithmetic is the
// fixed-order merge of bn_merge.hpp: mean = sum n_g mean_g / M, M2 = sum (M2_g + n_g (mean_g - mean)^2).
__global__ __launch_bounds__(THREADS) void records_merge_kernel(const float* __restrict__ records, int G, long rows_per_record,
                                                                long M, int C, float eps, float* __restrict__ stats) {
    __shared__ float red[THREADS];
    constexpr int CW = 4, SUB = THREADS / CW;
    const int cl = threadIdx.x % CW, sub = threadIdx.x / CW;
    const int c = blockIdx.x * CW + cl;
    float2 pv[8];
    float nn[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int g = sub + u * SUB;
        const int gc = min(g, G - 1);
        pv[u] = *reinterpret_cast<const float2*>(records + ((long)gc * C + c) * 2);
        const long lo = (long)gc * rows_per_record;
        nn[u] = g < G ? (float)(min(M, lo + rows_per_record) - lo) : 0.f;
    }
    float s_ = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) s_ = fmaf(nn[u], pv[u].x, s_);
    const float mean = bnm::reduce_sub(s_, red, CW) / (float)M;
    float m2 = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const float d = pv[u].x - mean;
        m2 += nn[u] > 0.f ? pv[u].y + nn[u] * d * d : 0.f;
    }
    m2 = bnm::reduce_sub(m2, red, CW);
    if (sub == 0) {
        stats[c] = mean;
        stats[C + c] = 1.0f / sqrtf(m2 / (float)M + eps);
    }
}

}  // namespace

// dst = conv(src) (+ add, element-wise, if add != NULL).  Returns -2 if the shape is not one of the
// specialised ones (the caller then uses the generic kernel).
int conv3x3_tiled(hipStream_t s, const float* src, const Filter3x3& w, const float* add, float* dst, float* bn_partial,
                   int N, int HW, int C, bool transposed) {
    if (C == 16 && HW == 32) return transposed ? launch<16, 32, 8, 1, 4, true>(s, src, w, add, dst, bn_partial, N) : launch<16, 32, 8, 1, 4, false>(s, src, w, add, dst, bn_partial, N);
    if (C == 32 && HW == 16) return transposed ? launch<32, 16, 8, 1, 4, true>(s, src, w, add, dst, bn_partial, N) : launch<32, 16, 8, 1, 4, false>(s, src, w, add, dst, bn_partial, N);
    if (C == 64 && HW == 8) return transposed ? launch<64, 8, 8, 2, 4, true>(s, src, w, add, dst, bn_partial, N) : launch<64, 8, 8, 2, 4, false>(s, src, w, add, dst, bn_partial, N);
    return -2;
}

// Forward convolution of a = ReLU(BN(src) (+ shortcut)), see PreBn.  in_parts: number of equal-sized
// statistics records of src in `records` (as emitted by the forward kernel for the same shape).
int conv3x3_tiled_prebn(hipStream_t s, const float* src, const float* records, int in_parts, const float* gamma,
                         const float* beta, float eps, const float* shortcut, bool half, float* act_out, float* stats_out,
                         const Filter3x3& w, float* dst, float* bn_partial, int N, int HW, int C) {
    PreBn pre;
    pre.half = half;
    pre.records = records;
    pre.M = (long)N * HW * HW;
    if (in_parts < 1 || pre.M % in_parts || in_parts > 32 * (THREADS / C)) return -1;
    pre.parts = in_parts;
    pre.rows = pre.M / in_parts;
    pre.gamma = gamma; pre.beta = beta; pre.eps = eps;
    pre.shortcut = shortcut; pre.act_out = act_out; pre.stats_out = stats_out;
    if (C != 16 && C != 32 && C != 64) return -2;
    if (in_parts > 8 * (THREADS / 4)) return -1;
    pre.merge = records_inline(in_parts, C);
    if (!pre.merge)
        hipLaunchKernelGGL(records_merge_kernel, dim3(C / 4), dim3(THREADS), 0, s, records, in_parts, pre.rows, pre.M, C, eps, stats_out);
    if (C == 16 && HW == 32)
        return shortcut ? launch<16, 32, 8, 1, 4, false, 2>(s, src, w, nullptr, dst, bn_partial, N, pre)
                        : launch<16, 32, 8, 1, 4, false, 1>(s, src, w, nullptr, dst, bn_partial, N, pre);
    if (C == 32 && HW == 16)
        return shortcut ? launch<32, 16, 8, 1, 4, false, 2>(s, src, w, nullptr, dst, bn_partial, N, pre)
                        : launch<32, 16, 8, 1, 4, false, 1>(s, src, w, nullptr, dst, bn_partial, N, pre);
    if (C == 64 && HW == 8)
        return shortcut ? launch<64, 8, 8, 2, 4, false, 2>(s, src, w, nullptr, dst, bn_partial, N, pre)
                        : launch<64, 8, 8, 2, 4, false, 1>(s, src, w, nullptr, dst, bn_partial, N, pre);
    return -2;
}

// d-input of the convolution (+ add) followed, in the same kernel, by the ReLU mask and the record sums of the
// batch norm that comes next in the backward direction, see PostBn.
int conv3x3_tiled_dgrad_post(hipStream_t s, const float* dy, const float* w, const float* add, float* dz,
                              const float* mask_src, const float* xc, const float* stats, float* records, int N, int HW, int C) {
    PostBn post{};
    post.mask_src = mask_src; post.xc = xc; post.stats = stats; post.records = records;
    if (C == 16 && HW == 32) return launch<16, 32, 8, 1, 4, true, 0, true>(s, dy, w, add, dz, nullptr, N, PreBn(), post);
    if (C == 32 && HW == 16) return launch<32, 16, 8, 1, 4, true, 0, true>(s, dy, w, add, dz, nullptr, N, PreBn(), post);
    if (C == 64 && HW == 8) return launch<64, 8, 8, 2, 4, true, 0, true>(s, dy, w, add, dz, nullptr, N, PreBn(), post);
    return -2;
}

// d-input convolution of dx = batch-norm backward of dz (see BwdBn), with the epilogue of conv3x3_tiled_dgrad_post;
// optionally carries the second stage of an earlier d-filter convolution (red_partial != NULL).
int conv3x3_tiled_dgrad_bn(hipStream_t s, const float* dz, const float* xc, const float* stats, const float* gamma,
                            const float* totals, const float* in_records, int parts, float* dgamma, float* dbeta, float* dx_out,
                            const Filter3x3& w, const float* add, float* out,
                            const float* mask_src, const float* xc_post, const float* stats_post, float* records,
                            const float* red_partial, float* red_dw, int red_E, int red_chunks, int N, int HW, int C,
                            const float* gamma_post, const float* beta_post) {
    if (!totals && !records_inline(parts, C)) return -1;
    BwdBn bwd;
    bwd.xc = xc; bwd.stats = stats; bwd.gamma = gamma; bwd.totals = totals; bwd.dx_out = dx_out;
    bwd.records = in_records; bwd.parts = parts; bwd.dgamma = dgamma; bwd.dbeta = dbeta;
    bwd.inv_m = 1.0f / (float)((long)N * HW * HW);
    PostBn post{};
    post.mask_src = mask_src; post.xc = xc_post; post.stats = stats_post; post.records = records; post.gamma = gamma_post; post.beta = beta_post;
    const jobs::ReduceJob rj = reduce_job({red_partial, red_dw, red_E, red_chunks, false}, THREADS);
    if (C == 16 && HW == 32) return launch<16, 32, 8, 1, 4, true, 3, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj);
    if (C == 32 && HW == 16) return launch<32, 16, 8, 1, 4, true, 3, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj);
    if (C == 64 && HW == 8) return launch<64, 8, 8, 2, 4, true, 3, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj);
    return -2;
}

// conv3x3_tiled_dgrad_bn with the d-filter convolution of the same layer in the same kernel (see WgradFused);
// dx is not stored.  Returns -2 for shapes the fused form does not cover (then the two-kernel form applies).
int conv3x3_tiled_dgrad_bn_wgrad(hipStream_t s, const float* dz, const float* xc, const float* stats, const float* gamma,
                                  const float* totals, const float* in_records, int parts, float* dgamma, float* dbeta,
                                  const Filter3x3& w, const float* add, float* out,
                                  const float* xc_post, const float* stats_post, float* records,
                                  const float* x_in, float* partial, const float* red_partial, float* red_dw, int red_E,
                                  int red_chunks, int N, int HW, int C, const float* gamma_post, const float* beta_post) {
    if (!totals && !records_inline(parts, C)) return -1;
    BwdBn bwd;
    bwd.xc = xc; bwd.stats = stats; bwd.gamma = gamma; bwd.totals = totals; bwd.dx_out = nullptr;
    bwd.records = in_records; bwd.parts = parts; bwd.dgamma = dgamma; bwd.dbeta = dbeta;
    bwd.inv_m = 1.0f / (float)((long)N * HW * HW);
    PostBn post{};
    post.mask_src = x_in; post.xc = xc_post; post.stats = stats_post; post.records = records; post.gamma = gamma_post; post.beta = beta_post;
    const jobs::ReduceJob rj = reduce_job({red_partial, red_dw, red_E, red_chunks, false}, THREADS);
    WgradFused wg;
    wg.x_in = x_in; wg.partial = partial;
    if (C == 16 && HW == 32) return launch<16, 32, 8, 1, 4, true, 3, true, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj, wg);
    if (C == 32 && HW == 16) return launch<32, 16, 8, 1, 4, true, 3, true, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj, wg);
    return -2;
}

bool conv3x3_records_inline(int parts, int C) { return records_inline(parts, C); }

// Number of per-workgroup statistics records (tiles of equal size) the forward kernel emits, 0 if the
// shape is not covered by it.
int conv3x3_tiled_stat_parts(int N, int HW, int C) {
    if (C == 16 && HW == 32) return N * 4;
    if (C == 32 && HW == 16) return N * 2;
    if (C == 64 && HW == 8) return N;
    return 0;
}

// ---------------------------------------------------------------------------------------------
// Gradient w.r.t. the filter of the same convolutions, stage 1 of 2: one workgroup per band of
// R rows of one image; the x halo tile and the dy tile sit in LDS and all nine taps
//   dw[tap][ci][co] += sum_{pixels of the band} x[pixel + tap][ci] * dy[pixel][co]
// are accumulated from them (x and dy are read from memory once), by minimal filtering (dfilter_run).  The
// matrix-core tile is 16 (ci) x 16 (co), the reduction runs over tiles of 2x2 pixels in runs of 16.
//   C = 16: one (ci, co) tile; the four wavefronts take one run each and are summed in a fixed order at the end.
//   C = 32: four (ci, co) tiles; wavefront w owns tile (w / 2, w % 2) and walks both runs.
// Output: partial[workgroup][tap][ci][co]; stage 2 (wgrad_reduce_kernel) sums over workgroups.
namespace {

template <int C, int HW, int R>
struct WCfg {
    static constexpr int LDC = C + 4;
    static constexpr int TW = HW + 2;
    static constexpr int XS = (R + 2) * TW * LDC;
    static constexpr int DS = R * HW * LDC;
    static constexpr bool SPLIT_K = (C == 16);
    static_assert(!SPLIT_K || (R / 2) * (HW / 2) == 64, "one run of 16 tiles per wavefront");
    static constexpr int RED = SPLIT_K ? 4 * 9 * C * C : 0;
    static constexpr size_t LDS_BYTES = (size_t)((XS + DS) > RED ? (XS + DS) : RED) * sizeof(float);
};

template <int C, int HW, int R>
__global__ __launch_bounds__(THREADS) void wgrad3x3_kernel(const float* __restrict__ x, const float* __restrict__ dy,
                                                           float* __restrict__ partial, int own_blocks, jobs::TotalsJob tj) {
    using K = WCfg<C, HW, R>;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    if ((int)blockIdx.x >= own_blocks) {            // workgroups behind the kernel's own carry the batch-norm sums job
        jobs::bn_totals(tj, blockIdx.x - own_blocks, lds);
        return;
    }
    float* Xs = lds;
    float* Ds = lds + K::XS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int BANDS = HW / R;
    const int tile = xcd_tile(blockIdx.x, own_blocks);
    const int band = tile % BANDS, n = tile / BANDS;
    const int r_base = band * R;
    constexpr int V = C / 4;
    for (int idx = tid; idx < (R + 2) * K::TW * V; idx += THREADS) {
        const int v = idx % V;
        const int pc = (idx / V) % K::TW, pr = idx / (V * K::TW);
        const int h = r_base + pr - 1, w = pc - 1;
        float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
        if (h >= 0 && h < HW && w >= 0 && w < HW)
            val = *reinterpret_cast<const float4*>(x + (((long)n * HW + h) * HW + w) * C + 4 * v);
        *reinterpret_cast<float4*>(&Xs[(pr * K::TW + pc) * K::LDC + 4 * v]) = val;
    }
    const float* dyb = dy + ((long)n * HW + r_base) * HW * C;
    for (int idx = tid; idx < R * HW * V; idx += THREADS) {
        const int v = idx % V, p = idx / V;
        *reinterpret_cast<float4*>(&Ds[p * K::LDC + 4 * v]) = *reinterpret_cast<const float4*>(dyb + (long)p * C + 4 * v);
    }
    __syncthreads();

    const int l16 = lane & 15, q = lane >> 4;
    const int cit = K::SPLIT_K ? 0 : wave >> 1, cot = K::SPLIT_K ? 0 : wave & 1;
    constexpr int TXN = HW / 2, WRUNS = (R / 2) * TXN / 16;
    floatx4 M[16];
#pragma unroll
    for (int xi = 0; xi < 16; ++xi) M[xi] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int run = K::SPLIT_K ? wave : 0; run < WRUNS; run += K::SPLIT_K ? 4 : 1) {
        dfilter_run(M, q,
                    [&](int tile) { return make_int2(2 * ((run * 16 + tile) / TXN), 2 * ((run * 16 + tile) % TXN)); },
                    [&](int2 o, int r, int c) { return Xs[((o.x + r) * K::TW + o.y + c) * K::LDC + 16 * cit + l16]; },
                    [&](int2 o, int i, int j) { return Ds[((o.x + i) * HW + o.y + j) * K::LDC + 16 * cot + l16]; });
    }
    mma::drain();
    floatx4 acc[9];
    dfilter_finish(M, acc);
    float* out = partial + (long)tile * 9 * C * C;
    if constexpr (K::SPLIT_K) {
        __syncthreads();                              // tiles no longer needed: reuse LDS for the 4 partial sums
        float* Red = lds;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) Red[wave * 9 * C * C + (t * C + 4 * q + v) * C + l16] = acc[t][v];
        __syncthreads();
        for (int idx = tid; idx < 9 * C * C; idx += THREADS)
            out[idx] = (Red[idx] + Red[9 * C * C + idx]) + (Red[2 * 9 * C * C + idx] + Red[3 * 9 * C * C + idx]);
    } else {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) out[(t * C + 16 * cit + 4 * q + v) * C + 16 * cot + l16] = acc[t][v];
    }
}

// The same for the last stage (64 channels, 8x8 images), on the bf16 matrix cores (split.hpp).  The result is as large as
// 9 x 64 x 64, so a workgroup owns 16 input and 32 output channels of it and four images, one per wavefront, which needs no
// barrier until the four sums meet in LDS: pixels are the reduction index, four image rows to an MFMA.  The wavefront leaves its
// slice of x (with a zero border) in LDS as three bf16 terms and takes it from there once per tap by transposing reads, the dy
// operands come straight from memory, eight pixels of a channel to a lane (through LDS too, 95 KB, two more kernels' workgroups
// would not fit beside: 10.2 us alone and 2 % of a ResNet step lost).  32 output channels (and not 16 of them and eight
// images) so that an x operand serves two products; rows of the matrix-core tile: co, columns: ci.  Output: partial[image group][tap][ci][co], 4.7 MB at batch 128 (as minimal filtering on the
// fp32 matrix cores, two images to a workgroup, 9.4 MB, each written and read once).
namespace wide {
constexpr int C = 64, HW = 8, TW = HW + 2, IMGS = 4, CI = 16, CO = 32;
constexpr int XPLANE = 2 * CI, XPITCH = 3 * XPLANE + 8;
constexpr int XB = TW * TW * XPITCH, RED = 2 * 9 * CI * CO * 4, LDS = 4 * XB > RED ? 4 * XB : RED;
static_assert(XB % 16 == 0, "alignment");
}  // namespace wide

__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2))) void wgrad3x3_wide_kernel(
    const float* __restrict__ x, const float* __restrict__ dy, float* __restrict__ partial, int N, int own_blocks, jobs::TotalsJob tj) {
    using namespace wide;
    extern __shared__ __attribute__((aligned(16))) char lds_bytes[];
    char* lds = lds_bytes;
    if ((int)blockIdx.x >= own_blocks) {
        jobs::bn_totals(tj, blockIdx.x - own_blocks, reinterpret_cast<float*>(lds));
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, q = lane >> 4;
    const int tile = xcd_tile(blockIdx.x, own_blocks);
    constexpr int ROLES = (C / CI) * (C / CO);
    const int role = tile % ROLES, grp = tile / ROLES, ci0 = CI * (role % (C / CI)), co0 = CO * (role / (C / CI));
    const int n = grp * IMGS + wave;
    char* X = lds + wave * XB;
    floatx4 acc[9][2];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t][0] = acc[t][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (n < N) {
        constexpr int NX = HW * HW * CI / 4 / 64;
        float4 rx[NX], rd[2][2][2];            // rd[run][co tile]: pixels 8 q .. 8 q + 7 of the run
#pragma unroll
        for (int e = 0; e < NX; ++e) {
            const int idx = lane + 64 * e;
            rx[e] = *reinterpret_cast<const float4*>(x + ((long)n * HW * HW + idx / (CI / 4)) * C + ci0 + 4 * (idx % (CI / 4)));
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float* dp = dy + ((long)n * HW * HW + 32 * r + 8 * q + 4 * e) * C + co0 + 16 * j + l16;
                    rd[r][j][e] = make_float4(dp[0], dp[C], dp[2 * C], dp[3 * C]);
                }
        for (int i = lane; i < 4 * (TW - 1) * (XPITCH / 8); i += 64) {          // zero border
            const int h = i / (XPITCH / 8);
            const int r = h < TW ? 0 : h < 2 * TW ? TW - 1 : (h - 2 * TW) / 2 + 1;
            const int c = h < 2 * TW ? h % TW : (h & 1) * (TW - 1);
            *reinterpret_cast<uint2*>(X + (r * TW + c) * XPITCH + 8 * (i % (XPITCH / 8))) = make_uint2(0u, 0u);
        }
        uint2 pl[split::PLANES];
#pragma unroll
        for (int e = 0; e < NX; ++e) {
            const int idx = lane + 64 * e, px = idx / (CI / 4);
            split::split4(split::scaled(rx[e]), pl);
#pragma unroll
            for (int p = 0; p < split::PLANES; ++p)
                *reinterpret_cast<uint2*>(X + ((px / HW + 1) * TW + px % HW + 1) * XPITCH + p * XPLANE + 8 * (idx % (CI / 4))) = pl[p];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const char* xa[2];                          // of pixels 8 q + 4 h + l16 / 4 of the first run (four rows)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int p = 8 * q + 4 * h + (l16 >> 2);
            xa[h] = X + (p / HW * TW + p % HW) * XPITCH + 8 * (l16 & 3);
        }
        split::Filt<32> d[2];
        uint4 xv[2][1][split::PLANES];
        auto load_x = [&](int i) {                  // run i / 9, tap i % 9
            const int off = ((4 * (i / 9) + i % 9 / 3) * TW + i % 3) * XPITCH;
            split::transposed_operand<XPLANE>(xv[i & 1][0], xa[0] + off, xa[1] + off);
        };
        load_x(0);
#pragma unroll
        for (int i = 0; i < 18; ++i) {
            if (i % 9 == 0)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) rd[i / 9][j][e] = split::scaled(rd[i / 9][j][e]);
                    d[j] = split::filter_operand<32>(rd[i / 9][j]);
                }
            if (i + 1 < 18) load_x(i + 1);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int PD[6] = {0, 2, 1, 0, 1, 0}, PX[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i % 9][j] = split::mfma(d[j].v[PD[p]], xv[i & 1][0][PX[p]], acc[i % 9][j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        mma::drain();
        float bad = 0.f;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j) bad = split::spoil(acc[t][j], bad);
        if (split::spoiled(bad)) {                  // beyond the range of the scaled terms: from the operands in memory, four pixels a step
#pragma unroll
            for (int t = 0; t < 9; ++t) acc[t][0] = acc[t][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int p = q; p < HW * HW; p += 4) {
                const float* dp = dy + ((long)n * HW * HW + p) * C + co0 + l16;
                const float d0[1] = {dp[0]}, d1[1] = {dp[16]};
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const int xh = p / HW + t / 3 - 1, xw = p % HW + t % 3 - 1;
                    const bool in = (unsigned)xh < (unsigned)HW && (unsigned)xw < (unsigned)HW;
                    const float xs[1] = {in ? x[(((long)n * HW + xh) * HW + xw) * C + ci0 + l16] : 0.f};
                    acc[t][0] = split::product32(d0, xs, acc[t][0]);
                    acc[t][1] = split::product32(d1, xs, acc[t][1]);
                }
            }
            mma::drain();
        } else {
#pragma unroll
            for (int t = 0; t < 9; ++t) { acc[t][0] *= split::UNSCALE; acc[t][1] *= split::UNSCALE; }
        }
    }
    // the four sums, in a fixed order: wavefronts 2 and 3 hand theirs to 0 and 1, those two meet in LDS
    floatx4* Red = reinterpret_cast<floatx4*>(lds); // [2][tap][ci][co / 4]
    constexpr int E4 = 9 * CI * CO / 4;
    floatx4* mine = Red + (wave & 1) * E4 + l16 * (CO / 4) + q;
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        __syncthreads();
        if (wave >> 1 == 1 - round)
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int j = 0; j < 2; ++j) mine[t * CI * (CO / 4) + 4 * j] = acc[t][j];
        __syncthreads();
        if (round == 0 && wave < 2)
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[t][j] += mine[t * CI * (CO / 4) + 4 * j];
    }
    float* out = partial + (long)grp * 9 * C * C;
    for (int idx = tid; idx < E4; idx += THREADS) {
        const int c4 = idx % (CO / 4), ci = idx / (CO / 4) % CI, t = idx / (CO / 4) / CI;
        *reinterpret_cast<floatx4*>(out + (t * C + ci0 + ci) * C + co0 + 4 * c4) = Red[idx] + Red[E4 + idx];
    }
}

int launch_wgrad_wide(hipStream_t s, const float* x, const float* dy, float* partial, int N, const jobs::TotalsJob& tj) {
    static_assert(wide::LDS >= jobs::LDS_FLOATS * sizeof(float), "room for a carried job");
    static bool attr_set = false;
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(wgrad3x3_wide_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, wide::LDS) !=
            hipSuccess)
            return -1;
        attr_set = true;
    }
    const int own = (N + wide::IMGS - 1) / wide::IMGS * (wide::C / wide::CI) * (wide::C / wide::CO);
    hipLaunchKernelGGL(wgrad3x3_wide_kernel, dim3(own + tj.blocks), dim3(THREADS), wide::LDS, s, x, dy, partial, N, own, tj);
    return DSSPK_LAUNCH_RC();
}

template <int C, int HW, int R>
int launch_wgrad(hipStream_t s, const float* x, const float* dy, float* partial, int N, const jobs::TotalsJob& tj) {
    using K = WCfg<C, HW, R>;
    static_assert(K::LDS_BYTES >= jobs::LDS_FLOATS * sizeof(float), "room for a carried job");
    static bool attr_set = false;
    auto kern = wgrad3x3_kernel<C, HW, R>;
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)K::LDS_BYTES) != hipSuccess)
            return -1;
        attr_set = true;
    }
    const int own = N * (HW / R);
    hipLaunchKernelGGL(kern, dim3(own + tj.blocks), dim3(THREADS), K::LDS_BYTES, s, x, dy, partial, own, tj);
    return DSSPK_LAUNCH_RC();
}

}  // namespace

// Number of partial results the specialised d-filter kernel writes, 0 if the shape is not covered.
int wgrad3x3_tiled_parts(int N, int HW, int C) {
    if (C == 16 && HW == 32) return N * 4;
    if (C == 32 && HW == 16) return N * 2;
    if (C == 64 && HW == 8) return (N + wide::IMGS - 1) / wide::IMGS;
    return 0;
}

int wgrad3x3_tiled(hipStream_t s, const float* x, const float* dy, float* partial, int N, int HW, int C, const jobs::TotalsJob& tj) {
    if (C == 16 && HW == 32) return launch_wgrad<16, 32, 8>(s, x, dy, partial, N, tj);
    if (C == 32 && HW == 16) return launch_wgrad<32, 16, 8>(s, x, dy, partial, N, tj);
    if (C == 64 && HW == 8) return launch_wgrad_wide(s, x, dy, partial, N, tj);
    return -2;
}
