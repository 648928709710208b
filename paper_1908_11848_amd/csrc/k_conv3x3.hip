// 3x3, stride 1, pad 1 convolutions with Cin = Cout = C (the 106 inner convolutions of
// ResNet-110): forward and gradient w.r.t. the input as ONE kernel.
//
// A workgroup owns a band of R output rows of one image (the whole 8x8 image in the last
// stage) and CN of the C output channels.  It loads the (R+2) x (HW+2) x C input halo tile
// (zero borders) into LDS once; everything else is served from LDS, so every input element
// is read from memory once per band instead of nine times.  The filter never passes through
// LDS: a wavefront owns ONE tile of 16 output channels and holds one column of that tile's filter
// (three taps) in registers, the next one being on its way.  LDS therefore holds the halo tile only (36 to
// 42 KB), registers stay below 128 (C = 16) or 170, and the workgroups of three or four kernels share a compute
// unit: one stream's transfers run beside another's products (with the whole filter in registers and two tiles in
// LDS for the fused d-filter, two: ResNet-110 at batch 128, 8 workers, 2.31 ms per push against 2.15).
//
// The arithmetic is fp32 on the bf16 matrix cores (split.hpp): the loader leaves every element in LDS as three bf16 terms
// (each converted once, not once per tap), the filter values are split in registers while the input is on its way, and six
// of the nine products are taken.  The matrix-core tile is 16 output channels (rows) x 16 pixels (columns); a wavefront owns
// one channel tile and four pixel tiles that lie below each other, so a pixel operand fetched for one filter row serves
// the tiles above it too, and a lane ends up with four consecutive channels of a pixel (16-byte loads and stores in the
// epilogue).
//
// Gradient w.r.t. the input of such a convolution is the same operation on dy with the filter
// taps reversed and its two channel indices swapped; only the filter fetch differs.
#include "mma.hpp"
#include "split.hpp"
#include "bn_merge.hpp"
#include "jobs.hpp"
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

template <int C, int HW, int R, int NSPLIT>
struct Cfg {
    static constexpr int CN = C / NSPLIT;          // output channels per workgroup
    static constexpr int PLANE = 2 * C;            // bytes between the three bf16 terms of a pixel in LDS
    // pitch of a pixel: 26 words (C = 16, 8-byte reads), 20 and 4 words (mod 32) for 16-byte reads, so that the operand reads of 16
    // pixels side by side meet 32 banks equally.  That is reckoned for these reads alone: with the staging stores and the d-filter's
    // transposing reads a quarter to a half of these kernels' LDS cycles are conflicts by the counters.
    static constexpr int PITCH = 3 * PLANE + (C == 16 ? 8 : 16);
    static constexpr int TW = HW + 2;              // halo tile width
    static constexpr int XB = (R + 2) * TW * PITCH;            // bytes
    static constexpr int WAVES_N = CN / 16;        // wavefronts side by side over the output channels
    static constexpr int WAVES_M = 4 / WAVES_N;    // ... and over the pixels or, in the last stage, the input channels
    // A wavefront works on four pixel tiles, each one (HW >= 16) or two (HW = 8) image rows below the one before.
    static constexpr int TROWS = HW >= 16 ? 1 : 2;
    static constexpr int TX = HW >= 16 ? HW / 16 : 1;          // tiles side by side
    static constexpr int WPX = R / (4 * TROWS) * TX;           // wavefronts over the band's pixels
    static constexpr int KS = WAVES_M / WPX;       // wavefronts that share pixels and split the input channels; they swap
                                                   // halves of their sums through LDS and each finishes its half
    static constexpr int WM = 4 / KS;              // pixel tiles a wavefront finishes
    static constexpr int SS = 8 * CN;              // floats: per-wavefront column sums (batch-norm records, two components)
    static constexpr int PS = 5 * C;               // floats: per-channel vectors of the loader
    static constexpr size_t LDS_BYTES = XB + (size_t)(SS + PS) * sizeof(float);
    // fused d-filter: the x halo tile takes the place of the first one; C = 16: four partial sums at the end
    static constexpr size_t RED = C == 16 ? 4 * 9 * C * C * sizeof(float) : 0;
    static constexpr size_t LDS_BYTES_WG = LDS_BYTES > RED ? LDS_BYTES : RED;
    static_assert(WPX * KS == WAVES_M && (KS == 1 || KS == 2) && (C == 16 || C == 32 * KS), "roles of the four wavefronts");
    static_assert(XB % 16 == 0 && KS * 4 * 4 * 64 * 16 / 2 <= XB, "alignment; room for the exchange");
};

// Normalisation applied to the input while it is loaded (PRE != 0): the kernel then computes
//   a = ReLU(gamma * (src - mean) * invstd + beta (+ shortcut))   and   dst = conv(a),
// i.e. the batch norm + ReLU that separates two convolutions never runs as a pass of its own.
// mean / invstd come from the statistics records of src, merged by a small kernel launched just before or, if they are few
// (records_inline), by every workgroup itself; they are also what the backward pass needs.  The workgroups write `a` (their own rows).
struct PreBn {
    const float* records;      // statistics records of src
    bnm::BnLayout L;           // their layout
    long M;                    // rows of src (= N * HW * HW)
    const float* gamma;
    const float* beta;
    float eps;
    const float* shortcut;     // PRE == 2: added before the ReLU, same shape as src
    float* act_out;            // a
    float* stats_out;          // mean[C], invstd[C]
    bool merge;                // every workgroup merges the records, the first one stores stats_out
};

// Backward of the ReLU + batch norm that FOLLOWS in the backward direction, started in the epilogue (POST):
// the result r (gradient w.r.t. a post-ReLU activation) is masked, dz = r * [mask_src > 0], dz is what gets
// stored, and the per-tile sums (sum dz, sum dz * xhat) with xhat = (xc - mean) * invstd are written as
// records for the batch norm's dx kernel.  This replaces that batch norm's stand-alone reduction pass.
struct PostBn {
    const float* mask_src;     // the saved post-ReLU activation
    const float* xc;           // the batch norm's input (convolution output)
    const float* stats;        // its mean[C], invstd[C]
    float* records;            // out: (sum dz, sum dz * xhat) per tile and channel
};

// Batch-norm backward applied to the input while it is loaded (PRE == 3, d-input convolutions): src is dz, the
// masked gradient at the batch norm's output, and the convolution runs on
//   dx = gamma * invstd * (dz - sum(dz) / M - xhat * sum(dz * xhat) / M),   xhat = (xc - mean) * invstd,
// the gradient w.r.t. the batch norm's input xc; the workgroups also write dx (their own rows) for the
// d-filter kernel.  The two sums come from the records of the epilogue that produced dz: added up before (TotalsJob) or, if
// they are few, by every workgroup itself.
struct BwdBn {
    const float* xc;           // the batch norm's input
    const float* stats;        // its mean[C], invstd[C]
    const float* gamma;
    const float* totals;       // sum dz [C], sum dz * xhat [C]; null: add up `records`
    const float* records;      // [parts][C][2]
    int parts;
    float *dgamma, *dbeta;     // with records: sum dz * xhat and sum dz, stored by the first workgroup
    float inv_m;               // 1 / (N * HW * HW)
    float* dx_out;
};

// Gradient w.r.t. the filter in the same kernel (WG, only with PRE == 3 and all channels in one workgroup): the
// dx tile the loader has just built in LDS is the d-filter convolution's dy, so only the convolution's input x
// (halo tile, a second LDS buffer) has to be fetched; dx itself never goes to memory.  After the d-input MFMA
// loop the wavefronts accumulate, as wgrad3x3_kernel does, dw[tap][ci][co] += x[pixel + tap][ci] * dx[pixel][co]
// over the band's pixels and store the workgroup's partial result; the sum over workgroups is a carried job of
// a later kernel.
struct WgradFused {
    const float* x_in;         // input of the convolution (post-ReLU activation of the layer below); it is also the
                               // source of the epilogue's ReLU mask, which is then taken from the LDS tile
    float* partial;            // out: [workgroup][9][C][C]
};

// add and dst may be the same buffer (every element is read and written by the same lane); with PRE == 3
// dst must differ from src, whose halo rows other workgroups still read.
// Wavefronts per SIMD the register allocation aims at: 4 (128 registers) fit the 16-channel kernels, 3 (168) the others; with 4 there
// the compiler spills up to 20.
template <int C, bool WG>
constexpr int min_waves() { return C == 16 && !WG ? 4 : 3; }

// Sum over the 16 lanes of a quarter wavefront, in all of them.
__device__ __forceinline__ float sum16(float v) {
#define ROR(n) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + n, 0xf, 0xf, true))
    v += ROR(8); v += ROR(4); v += ROR(2); v += ROR(1);
#undef ROR
    return v;
}
__device__ __forceinline__ float4 sum16(float4 v) { return make_float4(sum16(v.x), sum16(v.y), sum16(v.z), sum16(v.w)); }

// Records of a tensor small enough for every workgroup of its consumer to merge them itself, INLINE_RECORDS / C of them at most, so
// up to batch 32.  A kernel of its own for that takes 4 us of a stream's time.  20-layer network, four workers, a round with such
// kernels and without: batch 16 876 -> 821 us, batch 32 945 -> 894 us.  Twice as many would still win at batch 64 (1135 -> 1103 us),
// but their loads cost the smaller batches 2 % and, at four wavefronts a SIMD, spilled registers of the 16-channel kernels at every batch.
constexpr int INLINE_RECORDS = 2048, RECORDS_PER_THREAD = INLINE_RECORDS / THREADS;
constexpr bool records_inline(int parts, int C) { return (C == 16 || C == 32 || C == 64) && parts >= 1 && (long)parts * C <= INLINE_RECORDS; }

// Thread (channel tid % C, lane tid / C) holds records lane, lane + 256 / C, ... of its channel; all loads in flight together.
template <int C>
__device__ __forceinline__ void load_records(float2 (&v)[RECORDS_PER_THREAD], const float* __restrict__ records, int parts, int tid) {
#pragma unroll
    for (int u = 0; u < RECORDS_PER_THREAD; ++u) {
        const int g = tid / C + u * (THREADS / C);
        v[u] = *reinterpret_cast<const float2*>(records + ((long)min(g, parts - 1) * C + tid % C) * 2);
        if (g >= parts) v[u] = make_float2(0.f, 0.f);
    }
}

// Sum of every lane's s of this thread's channel, in lane order; red: THREADS floats nobody else uses between the barriers.
template <int C>
__device__ __forceinline__ float channel_sum(float s, float* red, int tid) {
    red[tid] = s;
    __syncthreads();
    float t = red[tid % C];
#pragma unroll
    for (int j = 1; j < THREADS / C; ++j) t += red[j * C + tid % C];
    return t;
}

template <int C, int HW, int R, int NSPLIT, bool TRANSPOSED, int PRE, bool POST = false, bool WG = false>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(min_waves<C, WG>()))) void conv3x3_kernel(const float* __restrict__ src, const float* __restrict__ wgt,
                                                          const float* add, float* dst,
                                                          float* __restrict__ bn_partial, PreBn pre, PostBn post, BwdBn bwd,
                                                          int conv_blocks, jobs::ReduceJob rj, WgradFused wg) {
    using K = Cfg<C, HW, R, NSPLIT>;
    static_assert(!WG || (PRE == 3 && NSPLIT == 1 && TRANSPOSED && (C == 16 || C == 32)), "fused d-filter: d-input form, whole channel range");
    extern __shared__ __attribute__((aligned(16))) char lds_bytes[];
    char* lds = lds_bytes;
    if ((int)blockIdx.x >= conv_blocks) {           // workgroups behind the convolution's own carry the reduction job
        jobs::wgrad_reduce(rj, blockIdx.x - conv_blocks, reinterpret_cast<float*>(lds));
        return;
    }
    char* Xs = lds;
    float* Ss = reinterpret_cast<float*>(lds + K::XB);          // column sums
    float* Sh = Ss + K::SS;                                     // per-channel vectors of the loader
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, q = lane >> 4;
    const int wave_n = wave % K::WAVES_N, wave_m = wave / K::WAVES_N;
    constexpr int BANDS = HW / R;
    const int tile = xcd_tile(blockIdx.x, conv_blocks);
    const int part = tile % NSPLIT;
    const int band = (tile / NSPLIT) % BANDS;
    const int n = tile / (NSPLIT * BANDS);
    const int r_base = band * R;                    // first output row of the band
    const int co_w = part * K::CN + 16 * wave_n;   // first output channel of this wavefront
    const int wpx = wave_m / K::KS, ks = wave_m % K::KS;       // its pixels, its share of the input channels
    const int row0 = wpx / K::TX * 4 * K::TROWS + (K::TROWS == 2 ? l16 >> 3 : 0);      // this lane's pixel in the first tile
    const int col = K::TROWS == 2 ? l16 & 7 : 16 * (wpx % K::TX) + l16;

    // ---- filter values of this lane, result channel co_w + l16 (row of the MFMA tile) and reduction channels k0 ..:
    //      forward : w[tap][k][co]           (C floats apart)
    //      d-input : w[8 - tap][co][k]       (16-byte loads, taps reversed)
    //      One filter column at a time (three taps): the product loop walks the columns, and the next one is on its way while it works
    //      on the present one.
    constexpr int FV = C == 16 ? 1 : 2;
    const int k0 = C == 16 ? 4 * q : 32 * ks + 8 * q;
    float4 fr[3][FV];
    auto load_filter = [&](int kx) {
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int e = 0; e < FV; ++e) {
                const int tap = 3 * ky + kx;
                if constexpr (TRANSPOSED) {
                    fr[ky][e] = *reinterpret_cast<const float4*>(wgt + ((long)(8 - tap) * C + co_w + l16) * C + k0 + 4 * e);
                } else {
                    const float* wp = wgt + ((long)tap * C + k0 + 4 * e) * C + co_w + l16;
                    fr[ky][e] = make_float4(wp[0], wp[C], wp[2 * C], wp[3 * C]);
                }
            }
    };
    float2 rec[PRE ? RECORDS_PER_THREAD : 1];
    if constexpr (PRE == 1 || PRE == 2)
        if (pre.merge) load_records<C>(rec, pre.records, pre.L.G, tid);
    if constexpr (PRE == 3)
        if (!bwd.totals) load_records<C>(rec, bwd.records, bwd.parts, tid);
    load_filter(0);
    // ---- input halo tile, zero outside the image.  The raw loads are issued first; the first filter column is split while
    //      they are in flight.
    constexpr int V = C / 4;
    constexpr int NL = ((R + 2) * K::TW * V + THREADS - 1) / THREADS;
    float4 val[NL], scv[PRE >= 2 ? NL : 1];
    const split::Buffer image = split::buffer(src + (long)n * HW * HW * C, 4u * HW * HW * C);
#pragma unroll
    for (int e = 0; e < NL; ++e) {
        const int idx = tid + e * THREADS;
        const int v = idx % V;
        const int pc = (idx / V) % K::TW, pr = idx / (V * K::TW);
        const int h = r_base + pr - 1, w = pc - 1;
        if constexpr (PRE == 0) {
            // Nothing but the scaling comes between load and split: behind a branch the compiler moves it up to the load, and each load
            // waits for the one before (batch 8: 6.7 instead of 5.9 us).  The others come out 0.1 to 0.4 us slower in this form.
            const bool in = pr < R + 2 && (unsigned)h < (unsigned)HW && (unsigned)w < (unsigned)HW;
            val[e] = split::load4(image, in ? 4u * (unsigned)((h * HW + w) * C + 4 * v) : split::OUTSIDE);
            continue;
        }
        val[e] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (pr < R + 2 && h >= 0 && h < HW && w >= 0 && w < HW) {
            const long off = (((long)n * HW + h) * HW + w) * C + 4 * v;
            val[e] = *reinterpret_cast<const float4*>(src + off);
            if constexpr (PRE == 2) scv[e] = *reinterpret_cast<const float4*>(pre.shortcut + off);
            if constexpr (PRE == 3) scv[e] = *reinterpret_cast<const float4*>(bwd.xc + off);
        }
    }
    split::Filt<C> filt[3];
    auto split_filter = [&]() {
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
#pragma unroll
            for (int e = 0; e < FV; ++e) fr[ky][e] = split::scaled(fr[ky][e]);
            filt[ky] = split::filter_operand<C>(fr[ky]);
        }
    };
    split_filter();
    float* red = reinterpret_cast<float*>(lds);         // the tile is not there yet
    if constexpr (PRE == 1 || PRE == 2) {               // mean / invstd of the input
        if (pre.merge) {                                // mean = sum n mean_g / M, M2 = sum (M2_g + n (mean_g - mean)^2)
            const float nn = (float)pre.L.rows_per_block, M = (float)pre.M;
            float s_ = 0.f, m2 = 0.f;
#pragma unroll
            for (int u = 0; u < RECORDS_PER_THREAD; ++u) s_ = fmaf(nn, rec[u].x, s_);
            const float mean = channel_sum<C>(s_, red, tid) / M;
#pragma unroll
            for (int u = 0; u < RECORDS_PER_THREAD; ++u) {
                const float d = rec[u].x - mean;
                m2 += tid / C + u * (THREADS / C) < pre.L.G ? rec[u].y + nn * d * d : 0.f;
            }
            const float invstd = 1.0f / sqrtf(channel_sum<C>(m2, red + THREADS, tid) / M + pre.eps);
            if (tid < C) {
                Sh[tid] = mean;
                Sh[C + tid] = invstd;
                if (blockIdx.x == 0) { pre.stats_out[tid] = mean; pre.stats_out[C + tid] = invstd; }
            }
        } else if (tid < 2 * C) {
            Sh[tid] = pre.stats_out[tid];
        }
        __syncthreads();
    }
    if constexpr (PRE == 3) {               // mean, invstd, gamma * invstd, sum(dz) / M, sum(dz * xhat) / M
        float sum_b = 0.f, sum_g = 0.f;
        if (!bwd.totals) {
#pragma unroll
            for (int u = 0; u < RECORDS_PER_THREAD; ++u) { sum_b += rec[u].x; sum_g += rec[u].y; }
            sum_b = channel_sum<C>(sum_b, red, tid);
            sum_g = channel_sum<C>(sum_g, red + THREADS, tid);
        } else if (tid < C) {
            sum_b = bwd.totals[tid];
            sum_g = bwd.totals[C + tid];
        }
        if (tid < C) {
            const float is = bwd.stats[C + tid];
            Sh[tid] = bwd.stats[tid];
            Sh[C + tid] = is;
            Sh[2 * C + tid] = bwd.gamma[tid] * is;
            Sh[3 * C + tid] = sum_b * bwd.inv_m;
            Sh[4 * C + tid] = sum_g * bwd.inv_m;
            if (!bwd.totals && blockIdx.x == 0) { bwd.dbeta[tid] = sum_b; bwd.dgamma[tid] = sum_g; }
        }
        __syncthreads();
    }
    auto stage = [&](char* to, float4 v) {  // 4 channels of a pixel as their three terms
        uint2 pl[split::PLANES];
        split::split4(split::scaled(v), pl);
#pragma unroll
        for (int p = 0; p < split::PLANES; ++p) *reinterpret_cast<uint2*>(to + p * K::PLANE) = pl[p];
    };
    // what the convolution runs on, four channels of a pixel of src (and of the shortcut or xc)
    auto transformed = [&](float4 o, float4 sc, int c) {
        if constexpr (PRE == 3) {
            const float4 mu = *reinterpret_cast<const float4*>(Sh + c);
            const float4 is = *reinterpret_cast<const float4*>(Sh + C + c);
            const float4 gi = *reinterpret_cast<const float4*>(Sh + 2 * C + c);
            const float4 db = *reinterpret_cast<const float4*>(Sh + 3 * C + c);
            const float4 dg = *reinterpret_cast<const float4*>(Sh + 4 * C + c);
            o.x = gi.x * (o.x - db.x - (sc.x - mu.x) * is.x * dg.x);
            o.y = gi.y * (o.y - db.y - (sc.y - mu.y) * is.y * dg.y);
            o.z = gi.z * (o.z - db.z - (sc.z - mu.z) * is.z * dg.z);
            o.w = gi.w * (o.w - db.w - (sc.w - mu.w) * is.w * dg.w);
        }
        if constexpr (PRE == 1 || PRE == 2) {
            const float4 mu = *reinterpret_cast<const float4*>(Sh + c);
            const float4 is = *reinterpret_cast<const float4*>(Sh + C + c);
            const float4 ga = *reinterpret_cast<const float4*>(pre.gamma + c);
            const float4 be = *reinterpret_cast<const float4*>(pre.beta + c);
            o.x = fmaf((o.x - mu.x) * is.x, ga.x, be.x);
            o.y = fmaf((o.y - mu.y) * is.y, ga.y, be.y);
            o.z = fmaf((o.z - mu.z) * is.z, ga.z, be.z);
            o.w = fmaf((o.w - mu.w) * is.w, ga.w, be.w);
            if constexpr (PRE == 2) { o.x += sc.x; o.y += sc.y; o.z += sc.z; o.w += sc.w; }
            o.x = fmaxf(o.x, 0.f); o.y = fmaxf(o.y, 0.f); o.z = fmaxf(o.z, 0.f); o.w = fmaxf(o.w, 0.f);
        }
        return o;
    };
    auto input = [&](int h, int w, int c) {  // the same from memory, zero outside the image
        if (h < 0 || h >= HW || w < 0 || w >= HW) return make_float4(0.f, 0.f, 0.f, 0.f);
        const long off = (((long)n * HW + h) * HW + w) * C + c;
        float4 sc = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (PRE == 2) sc = *reinterpret_cast<const float4*>(pre.shortcut + off);
        if constexpr (PRE == 3) sc = *reinterpret_cast<const float4*>(bwd.xc + off);
        return transformed(*reinterpret_cast<const float4*>(src + off), sc, c);
    };
#pragma unroll
    for (int e = 0; e < NL; ++e) {
        const int idx = tid + e * THREADS;
        const int v = idx % V;
        const int pc = (idx / V) % K::TW, pr = idx / (V * K::TW);
        const int h = r_base + pr - 1, w = pc - 1;
        if (pr >= R + 2) continue;
        if constexpr (PRE != 0) {
            if (h >= 0 && h < HW && w >= 0 && w < HW) {
                val[e] = transformed(val[e], scv[PRE >= 2 ? e : 0], 4 * v);
                // the band's own rows (not the halo rows) are this workgroup's part of `a` or dx
                if (!WG && part == 0 && pr >= 1 && pr <= R)
                    *reinterpret_cast<float4*>((PRE == 3 ? bwd.dx_out : pre.act_out) + (((long)n * HW + h) * HW + w) * C + 4 * v) = val[e];
            }
        }
        stage(Xs + (pr * K::TW + pc) * K::PITCH + 8 * v, val[e]);
    }
    load_filter(1);
    // x halo tile of the fused d-filter: on its way during the product loop (pixels outside the image: some other pixel, zeroed later)
    float4 xin[WG ? NL : 1];
    if constexpr (WG) {
#pragma unroll
        for (int e = 0; e < NL; ++e) {
            const int idx = tid + e * THREADS;
            const int v = idx % V, pc = (idx / V) % K::TW, pr = idx / (V * K::TW);
            const int h = min(max(r_base + pr - 1, 0), HW - 1), w = min(max(pc - 1, 0), HW - 1);
            xin[e] = *reinterpret_cast<const float4*>(wg.x_in + (((long)n * HW + h) * HW + w) * C + 4 * v);
        }
    }
    __syncthreads();

    // ---- products.  Pixel operand (st, kx): the tile that starts st rows below the wavefront's first one, kx to the right
    //      (halo coordinates); it meets filter row ky in the tile t with TROWS t + ky = st.
    floatx4 acc[K::WM];
    {
        constexpr int ST = 3 * K::TROWS + 3;
        const char* base = Xs + (row0 * K::TW + col) * K::PITCH + (C == 16 ? 8 : 16) * q + 64 * ks;
        // Two accumulators: the leading products, and the small ones (2^-8 and less of them), so that most of the roundings are
        // those of the small sum.
        floatx4 a[4], lo[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = lo[t] = floatx4{0.f, 0.f, 0.f, 0.f};
        split::Pix<C> x[2];
        auto pixels = [&](int i) { return split::pixel_operand<C, K::PLANE>(base + (i % ST * K::TW + i / ST) * K::PITCH); };
        x[0] = pixels(0);
#pragma unroll
        for (int i = 0; i < 3 * ST; ++i) {
            const int st = i % ST, kx = i / ST;
            if (kx > 0 && st == 0) {
                split_filter();
                if (kx == 1) load_filter(2);
            }
            if (i + 1 < 3 * ST) x[(i + 1) & 1] = pixels(i + 1);
            __builtin_amdgcn_sched_barrier(0);      // or the compiler moves the reads down to their use, behind the products
#pragma unroll
            for (int p = 0; p < split::products<C>(); ++p)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int ky = st - K::TROWS * t;
                    if (ky < 0 || ky > 2) continue;
                    floatx4& to = p + 1 < split::products<C>() ? lo[t] : a[t];
                    to = split::product<C>(p, filt[ky], x[i & 1], to);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        mma::drain();
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] += lo[t];
        if constexpr (K::KS == 1) {
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = a[t];
        } else {
            // the two wavefronts of a group of pixels hold partial sums over their halves of the input channels: each
            // hands the other the two tiles it will not finish and adds what it receives (first half + second half)
            __syncthreads();                               // every wavefront has read the tile for the last time
            float* Ex = reinterpret_cast<float*>(lds);             // [wavefront][2][64][4]
#pragma unroll
            for (int wm = 0; wm < 2; ++wm)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float give = ks == 0 ? a[2 + wm][v] : a[wm][v];
                    acc[wm][v] = ks == 0 ? a[wm][v] : a[2 + wm][v];
                    Ex[((wave * 2 + wm) * 64 + lane) * 4 + v] = give;
                }
            __syncthreads();
            const int partner = (wave_m ^ 1) * K::WAVES_N + wave_n;
#pragma unroll
            for (int wm = 0; wm < 2; ++wm)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[wm][v] += Ex[((partner * 2 + wm) * 64 + lane) * 4 + v];
        }
    }

    float bad = 0.f;
#pragma unroll
    for (int wm = 0; wm < K::WM; ++wm) bad = split::spoil(acc[wm], bad);
    if (split::spoiled(bad)) {      // beyond the range of the scaled terms: the wavefront's tiles from the operands in memory
#pragma unroll
        for (int wm = 0; wm < K::WM; ++wm) {
            acc[wm] = floatx4{0.f, 0.f, 0.f, 0.f};
            const int h0 = r_base + row0 + K::TROWS * (ks * K::WM + wm) - 1;
#pragma unroll 1
            for (int tap = 0; tap < 9; ++tap)
#pragma unroll 1
                for (int c = 4 * q; c < C; c += 16) {
                    const float4 x = input(h0 + tap / 3, col + tap % 3 - 1, c);
                    float4 y;
                    if constexpr (TRANSPOSED) {
                        y = *reinterpret_cast<const float4*>(wgt + ((long)(8 - tap) * C + co_w + l16) * C + c);
                    } else {
                        const float* wp = wgt + ((long)tap * C + c) * C + co_w + l16;
                        y = make_float4(wp[0], wp[C], wp[2 * C], wp[3 * C]);
                    }
                    const float a[4] = {y.x, y.y, y.z, y.w}, b[4] = {x.x, x.y, x.z, x.w};
                    acc[wm] = split::product32(a, b, acc[wm]);
                }
        }
        mma::drain();
    } else {
#pragma unroll
        for (int wm = 0; wm < K::WM; ++wm) acc[wm] *= split::UNSCALE;
    }

    // ---- store: a lane holds channels co .. co + 3 of its pixel of every tile
    const int co = co_w + 4 * q;
    float4 mu_c = make_float4(0.f, 0.f, 0.f, 0.f), is_c = mu_c;
    auto row_of = [&](int wm) { return row0 + K::TROWS * (ks * K::WM + wm); };
    auto out_off = [&](int wm) { return (((long)n * HW + r_base + row_of(wm)) * HW + col) * C + co; };
    // all loads of the epilogue together (dst may alias add, so the compiler cannot move them across the stores itself)
    float4 addv[K::WM], maskv[POST ? K::WM : 1], xcv[POST ? K::WM : 1];
    unsigned mask_bits = 0;         // WG: bit 4 wm + channel
    auto epilogue_loads = [&]() {
        if constexpr (POST) {
            mu_c = *reinterpret_cast<const float4*>(post.stats + co);
            is_c = *reinterpret_cast<const float4*>(post.stats + C + co);
        }
#pragma unroll
        for (int wm = 0; wm < K::WM; ++wm) {
            const long off = out_off(wm);
            addv[wm] = add ? *reinterpret_cast<const float4*>(add + off) : make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (POST) {
                if constexpr (!WG) maskv[wm] = *reinterpret_cast<const float4*>(post.mask_src + off);
                xcv[wm] = *reinterpret_cast<const float4*>(post.xc + off);
            }
        }
    };
    if constexpr (!WG) epilogue_loads();
    if constexpr (WG) {
        // ---- d-filter of the same layer:
        //      dw[tap][ci][co] += x[pixel + tap][ci] dx[pixel][co], pixels as reduction index, 32 to an MFMA, both operands
        //      by transposing reads.  The dx operands go to registers (the product loop is through with the tile), the x tile
        //      takes the place of the dx tile: half the LDS, so that workgroups of two more kernels fit beside this one's.
        //      A run of 32 pixels is one image row (C = 16) or two (C = 32); an x operand fetched
        //      for one filter row serves the run above it too.  Rows of the matrix-core tile: co, columns: ci.
        //      C = 16: one 16x16 tile of (ci, co); a wavefront takes two of the band's eight runs, the four are summed
        //      in a fixed order.  C = 32: wavefront w owns tile (w / 2, w % 2) and takes all four runs.
        constexpr bool SPLIT_K = (C == 16);
        constexpr int RROWS = 32 / HW, RUNS = SPLIT_K ? 2 : 4;     // image rows per run, runs per wavefront
        const int cit = SPLIT_K ? 0 : wave >> 1, cot = SPLIT_K ? 0 : wave & 1;
        const int first = SPLIT_K ? RUNS * wave : 0;               // first image row of the wavefront's runs
        const char* xa[2];                                         // of pixels 8 q + 4 h + l16 / 4 of the first run
        constexpr int ST = RROWS * (RUNS - 1) + 3;                 // image rows the runs and the three filter rows meet
        uint4 d[RUNS][split::PLANES], x[2][split::PLANES];
        {
            const char* da[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int p = 8 * q + 4 * h + (l16 >> 2);
                const int o = ((first + p / HW) * K::TW + p % HW) * K::PITCH + 8 * (l16 & 3);
                xa[h] = Xs + o + 32 * cit;
                da[h] = Xs + o + (K::TW + 1) * K::PITCH + 32 * cot;
            }
#pragma unroll
            for (int run = 0; run < RUNS; ++run)
                split::transposed_operand<K::PLANE>(d[run], da[0] + run * RROWS * K::TW * K::PITCH, da[1] + run * RROWS * K::TW * K::PITCH);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < NL; ++e) {
            const int idx = tid + e * THREADS;
            const int v = idx % V, pc = (idx / V) % K::TW, pr = idx / (V * K::TW);
            const int h = r_base + pr - 1, w = pc - 1;
            if (pr >= R + 2) continue;
            const bool in = h >= 0 && h < HW && w >= 0 && w < HW;
            stage(Xs + (pr * K::TW + pc) * K::PITCH + 8 * v,
                  make_float4(in ? xin[e].x : 0.f, in ? xin[e].y : 0.f, in ? xin[e].z : 0.f, in ? xin[e].w : 0.f));
        }
        __syncthreads();
#pragma unroll
        for (int wm = 0; wm < K::WM; ++wm) {        // the mask source is the convolution's input, whose leading terms are in LDS
            const uint2 m = *reinterpret_cast<const uint2*>(Xs + ((row_of(wm) + 1) * K::TW + col + 1) * K::PITCH + 2 * co);
            const float f[4] = {__uint_as_float(m.x << 16), __uint_as_float(m.x & 0xffff0000u), __uint_as_float(m.y << 16), __uint_as_float(m.y & 0xffff0000u)};
#pragma unroll
            for (int v = 0; v < 4; ++v) mask_bits |= f[v] > 0.f ? 1u << (4 * wm + v) : 0u;
        }
        // One filter column after the other, its small products with accumulators of their own: in one accumulator all six are rounded to
        // the size of the sum, and with a bias, so that the error of the sum over the workgroups grew with their number (16 channels,
        // batch 1 / 37 / 128: 1.1e-7 / 2.0e-7 / 3.2e-7; so 0.7e-7 / 1.0e-7 / 1.2e-7).
        floatx4 dw[9];
        auto load_x = [&](int b, int i) {
            const int off = (i % ST * K::TW + i / ST) * K::PITCH;
            split::transposed_operand<K::PLANE>(x[b], xa[0] + off, xa[1] + off);
        };
        load_x(0, 0);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            floatx4 lead[3], small[3];
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) lead[ky] = small[ky] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < ST; ++st) {
                const int i = ST * kx + st;
                if (i + 1 < 3 * ST) load_x((i + 1) & 1, i + 1);
                __builtin_amdgcn_sched_barrier(0);
                constexpr int PD[6] = {0, 2, 1, 0, 1, 0}, PX[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
                for (int p = 0; p < 6; ++p)
#pragma unroll
                    for (int run = 0; run < RUNS; ++run) {
                        const int ky = st - RROWS * run;
                        if (ky < 0 || ky > 2) continue;
                        floatx4& to = p < 5 ? small[ky] : lead[ky];
                        to = split::mfma(d[run][PD[p]], x[i & 1][PX[p]], to);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) dw[3 * ky + kx] = lead[ky] + small[ky];
        }
        float worst = 0.f;
#pragma unroll
        for (int t = 0; t < 9; ++t) worst = split::spoil(dw[t], worst);
        if (split::spoiled(worst)) {        // the wavefront's runs from the operands in memory, four pixels of a row a step
#pragma unroll
            for (int t = 0; t < 9; ++t) dw[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int p = first * HW + q; p < (first + RUNS * RROWS) * HW; p += 4) {
                const int h = r_base + p / HW, w = p % HW, c = 16 * cot + l16;
                const float4 dx = input(h, w, c & ~3);
                const float d[1] = {c & 2 ? (c & 1 ? dx.w : dx.z) : (c & 1 ? dx.y : dx.x)};
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const int xh = h + t / 3 - 1, xw = w + t % 3 - 1;
                    const bool in = (unsigned)xh < (unsigned)HW && (unsigned)xw < (unsigned)HW;
                    const float xv[1] = {in ? wg.x_in[(((long)n * HW + xh) * HW + xw) * C + 16 * cit + l16] : 0.f};
                    dw[t] = split::product32(d, xv, dw[t]);
                }
            }
            mma::drain();
        } else {
#pragma unroll
            for (int t = 0; t < 9; ++t) dw[t] *= split::UNSCALE;
        }
        epilogue_loads();
        float* pout = wg.partial + (long)tile * 9 * C * C;
        if constexpr (SPLIT_K) {
            static_assert(!SPLIT_K || 4 * 9 * C * C * sizeof(float) <= K::LDS_BYTES_WG, "room for the four partial sums");
            __syncthreads();                              // both tiles are no longer needed: reuse LDS for the 4 partial sums
            floatx4* Red = reinterpret_cast<floatx4*>(lds);       // [wavefront][tap][ci][co / 4]
            constexpr int E4 = 9 * C * C / 4;
#pragma unroll
            for (int t = 0; t < 9; ++t) Red[wave * E4 + (t * C + l16) * 4 + q] = dw[t];
            __syncthreads();
            for (int idx = tid; idx < E4; idx += THREADS)
                reinterpret_cast<floatx4*>(pout)[idx] = (Red[idx] + Red[E4 + idx]) + (Red[2 * E4 + idx] + Red[3 * E4 + idx]);
            __syncthreads();                              // before the epilogue's sums use LDS again
        } else {
#pragma unroll
            for (int t = 0; t < 9; ++t)
                *reinterpret_cast<floatx4*>(pout + (t * C + 16 * cit + l16) * C + 16 * cot + 4 * q) = dw[t];
        }
    }
    float4 sum_dz = make_float4(0.f, 0.f, 0.f, 0.f), sum_dzx = sum_dz;
#pragma unroll
    for (int wm = 0; wm < K::WM; ++wm) {
        float4 r = make_float4(acc[wm][0] + addv[wm].x, acc[wm][1] + addv[wm].y, acc[wm][2] + addv[wm].z, acc[wm][3] + addv[wm].w);
        if constexpr (POST) {
            auto on = [&](int v, float m) { return WG ? (mask_bits >> (4 * wm + v) & 1u) != 0 : m > 0.f; };
            r.x = on(0, maskv[wm].x) ? r.x : 0.f; r.y = on(1, maskv[wm].y) ? r.y : 0.f;
            r.z = on(2, maskv[wm].z) ? r.z : 0.f; r.w = on(3, maskv[wm].w) ? r.w : 0.f;
            sum_dz.x += r.x; sum_dz.y += r.y; sum_dz.z += r.z; sum_dz.w += r.w;
            sum_dzx.x = fmaf(r.x, (xcv[wm].x - mu_c.x) * is_c.x, sum_dzx.x);
            sum_dzx.y = fmaf(r.y, (xcv[wm].y - mu_c.y) * is_c.y, sum_dzx.y);
            sum_dzx.z = fmaf(r.z, (xcv[wm].z - mu_c.z) * is_c.z, sum_dzx.z);
            sum_dzx.w = fmaf(r.w, (xcv[wm].w - mu_c.w) * is_c.w, sum_dzx.w);
        }
        *reinterpret_cast<float4*>(dst + out_off(wm)) = r;
    }
    // per-channel totals over the workgroup's tile: lanes of a wavefront by lane rotations, then the WAVES_M
    // wavefronts that share the channel tile through LDS, in a fixed order
    const int cl = 16 * wave_n + 4 * q;              // first channel inside the workgroup's CN
    auto put = [&](float* S, float4 v) { if (l16 == 0) *reinterpret_cast<float4*>(S + wave_m * K::CN + cl) = v; };
    auto tile_total = [&](const float* S) {
        float4 t = *reinterpret_cast<const float4*>(S + cl);
#pragma unroll
        for (int m = 1; m < K::WAVES_M; ++m) {
            const float4 o = *reinterpret_cast<const float4*>(S + m * K::CN + cl);
            t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
        }
        return t;
    };
    auto put_records = [&](float* records, float4 a_, float4 b_) {      // pairs per channel
        float4* to = reinterpret_cast<float4*>(records + ((long)(n * BANDS + band) * C + co) * 2);
        to[0] = make_float4(a_.x, b_.x, a_.y, b_.y);
        to[1] = make_float4(a_.z, b_.z, a_.w, b_.w);
    };
    if constexpr (POST) {
        put(Ss, sum16(sum_dz));
        put(Ss + 4 * K::CN, sum16(sum_dzx));
        __syncthreads();
        if (wave_m == 0 && l16 == 0) put_records(post.records, tile_total(Ss), tile_total(Ss + 4 * K::CN));
    }

    // ---- optional: batch-norm statistics of this workgroup's output tile, per channel:
    //      mean over its R*HW pixels and the sum of squared deviations from that mean
    //      (bn_partial[(g*C + c)*2 + {0,1}], g = image * bands + band), merged later like row slabs.
    if (bn_partial) {
        constexpr float inv_n = 1.0f / (float)(R * HW);
        float4 mean = make_float4(0.f, 0.f, 0.f, 0.f), s_ = mean;
#pragma unroll
        for (int wm = 0; wm < K::WM; ++wm) { s_.x += acc[wm][0]; s_.y += acc[wm][1]; s_.z += acc[wm][2]; s_.w += acc[wm][3]; }
        put(Ss, sum16(s_));
        __syncthreads();
        mean = tile_total(Ss);
        mean.x *= inv_n; mean.y *= inv_n; mean.z *= inv_n; mean.w *= inv_n;
        s_ = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int wm = 0; wm < K::WM; ++wm) {
            const float dx = acc[wm][0] - mean.x, dy = acc[wm][1] - mean.y, dz = acc[wm][2] - mean.z, dw = acc[wm][3] - mean.w;
            s_.x += dx * dx; s_.y += dy * dy; s_.z += dz * dz; s_.w += dw * dw;
        }
        put(Ss + 4 * K::CN, sum16(s_));
        __syncthreads();
        if (wave_m == 0 && l16 == 0) put_records(bn_partial, mean, tile_total(Ss + 4 * K::CN));
    }
}

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
    const float mean = bnm::reduce_sub(s_, red, cl, sub, SUB, CW) / (float)M;
    float m2 = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const float d = pv[u].x - mean;
        m2 += nn[u] > 0.f ? pv[u].y + nn[u] * d * d : 0.f;
    }
    m2 = bnm::reduce_sub(m2, red, cl, sub, SUB, CW);
    if (sub == 0) {
        stats[c] = mean;
        stats[C + c] = 1.0f / sqrtf(m2 / (float)M + eps);
    }
}

template <int C, int HW, int R, int NSPLIT, bool T, int PRE = 0, bool POST = false, bool WG = false>
int launch(hipStream_t s, const float* src, const float* w, const float* add, float* dst, float* bn_partial, int N,
           const PreBn& pre = PreBn{}, const PostBn& post = PostBn(), const BwdBn& bwd = BwdBn(),
           const jobs::ReduceJob& rj = jobs::ReduceJob(), const WgradFused& wg = WgradFused()) {
    using K = Cfg<C, HW, R, NSPLIT>;
    constexpr size_t LDS_BYTES = WG ? K::LDS_BYTES_WG : K::LDS_BYTES;
    static_assert(LDS_BYTES >= jobs::LDS_FLOATS * sizeof(float), "room for a carried job");
    static bool attr_set = false;       // raise the dynamic-LDS limit once per instantiation
    auto kern = conv3x3_kernel<C, HW, R, NSPLIT, T, PRE, POST, WG>;
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)LDS_BYTES) != hipSuccess)
            return -1;
        attr_set = true;
    }
    const int conv_blocks = N * (HW / R) * NSPLIT;
    hipLaunchKernelGGL(kern, dim3(conv_blocks + rj.blocks), dim3(THREADS), LDS_BYTES, s, src, w, add, dst, bn_partial, pre, post,
                       bwd, conv_blocks, rj, wg);
    return DSSPK_LAUNCH_RC();
}

}  // namespace

// dst = conv(src) (+ add, element-wise, if add != NULL).  Returns -2 if the shape is not one of the
// specialised ones (the caller then uses the generic kernel).
int conv3x3_tiled(hipStream_t s, const float* src, const float* w, const float* add, float* dst, float* bn_partial,
                   int N, int HW, int C, bool transposed) {
    if (C == 16 && HW == 32) return transposed ? launch<16, 32, 8, 1, true>(s, src, w, add, dst, bn_partial, N) : launch<16, 32, 8, 1, false>(s, src, w, add, dst, bn_partial, N);
    if (C == 32 && HW == 16) return transposed ? launch<32, 16, 8, 1, true>(s, src, w, add, dst, bn_partial, N) : launch<32, 16, 8, 1, false>(s, src, w, add, dst, bn_partial, N);
    if (C == 64 && HW == 8) return transposed ? launch<64, 8, 8, 2, true>(s, src, w, add, dst, bn_partial, N) : launch<64, 8, 8, 2, false>(s, src, w, add, dst, bn_partial, N);
    return -2;
}

// Forward convolution of a = ReLU(BN(src) (+ shortcut)), see PreBn.  in_parts: number of equal-sized
// statistics records of src in `records` (as emitted by the forward kernel for the same shape).
int conv3x3_tiled_prebn(hipStream_t s, const float* src, const float* records, int in_parts, const float* gamma,
                         const float* beta, float eps, const float* shortcut, float* act_out, float* stats_out,
                         const float* w, float* dst, float* bn_partial, int N, int HW, int C) {
    PreBn pre;
    pre.records = records;
    pre.M = (long)N * HW * HW;
    if (in_parts < 1 || pre.M % in_parts || in_parts > 32 * (THREADS / C)) return -1;
    pre.L = bnm::bn_layout(pre.M, C);
    pre.L.G = in_parts;
    pre.L.rows_per_block = pre.M / in_parts;
    pre.gamma = gamma; pre.beta = beta; pre.eps = eps;
    pre.shortcut = shortcut; pre.act_out = act_out; pre.stats_out = stats_out;
    if (C != 16 && C != 32 && C != 64) return -2;
    if (in_parts > 8 * (THREADS / 4)) return -1;
    pre.merge = records_inline(in_parts, C);
    if (!pre.merge)
        hipLaunchKernelGGL(records_merge_kernel, dim3(C / 4), dim3(THREADS), 0, s, records, in_parts, pre.L.rows_per_block, pre.M, C, eps, stats_out);
    if (C == 16 && HW == 32)
        return shortcut ? launch<16, 32, 8, 1, false, 2>(s, src, w, nullptr, dst, bn_partial, N, pre)
                        : launch<16, 32, 8, 1, false, 1>(s, src, w, nullptr, dst, bn_partial, N, pre);
    if (C == 32 && HW == 16)
        return shortcut ? launch<32, 16, 8, 1, false, 2>(s, src, w, nullptr, dst, bn_partial, N, pre)
                        : launch<32, 16, 8, 1, false, 1>(s, src, w, nullptr, dst, bn_partial, N, pre);
    if (C == 64 && HW == 8)
        return shortcut ? launch<64, 8, 8, 2, false, 2>(s, src, w, nullptr, dst, bn_partial, N, pre)
                        : launch<64, 8, 8, 2, false, 1>(s, src, w, nullptr, dst, bn_partial, N, pre);
    return -2;
}

// d-input of the convolution (+ add) followed, in the same kernel, by the ReLU mask and the record sums of the
// batch norm that comes next in the backward direction, see PostBn.
int conv3x3_tiled_dgrad_post(hipStream_t s, const float* dy, const float* w, const float* add, float* dz,
                              const float* mask_src, const float* xc, const float* stats, float* records, int N, int HW, int C) {
    PostBn post;
    post.mask_src = mask_src; post.xc = xc; post.stats = stats; post.records = records;
    if (C == 16 && HW == 32) return launch<16, 32, 8, 1, true, 0, true>(s, dy, w, add, dz, nullptr, N, PreBn(), post);
    if (C == 32 && HW == 16) return launch<32, 16, 8, 1, true, 0, true>(s, dy, w, add, dz, nullptr, N, PreBn(), post);
    if (C == 64 && HW == 8) return launch<64, 8, 8, 2, true, 0, true>(s, dy, w, add, dz, nullptr, N, PreBn(), post);
    return -2;
}

// d-input convolution of dx = batch-norm backward of dz (see BwdBn), with the epilogue of conv3x3_tiled_dgrad_post;
// optionally carries the second stage of an earlier d-filter convolution (red_partial != NULL).
int conv3x3_tiled_dgrad_bn(hipStream_t s, const float* dz, const float* xc, const float* stats, const float* gamma,
                            const float* totals, const float* in_records, int parts, float* dgamma, float* dbeta, float* dx_out,
                            const float* w, const float* add, float* out,
                            const float* mask_src, const float* xc_post, const float* stats_post, float* records,
                            const float* red_partial, float* red_dw, int red_E, int red_chunks, int N, int HW, int C) {
    if (!totals && !records_inline(parts, C)) return -1;
    BwdBn bwd;
    bwd.xc = xc; bwd.stats = stats; bwd.gamma = gamma; bwd.totals = totals; bwd.dx_out = dx_out;
    bwd.records = in_records; bwd.parts = parts; bwd.dgamma = dgamma; bwd.dbeta = dbeta;
    bwd.inv_m = 1.0f / (float)((long)N * HW * HW);
    PostBn post;
    post.mask_src = mask_src; post.xc = xc_post; post.stats = stats_post; post.records = records;
    jobs::ReduceJob rj = jobs::ReduceJob();
    if (red_partial) {
        rj.partial = red_partial; rj.dw = red_dw; rj.E = red_E; rj.chunks = red_chunks;
        const int groups = jobs::reduce_groups(red_E, red_chunks);
        rj.blocks = groups < 288 ? groups : 288;
    }
    if (C == 16 && HW == 32) return launch<16, 32, 8, 1, true, 3, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj);
    if (C == 32 && HW == 16) return launch<32, 16, 8, 1, true, 3, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj);
    if (C == 64 && HW == 8) return launch<64, 8, 8, 2, true, 3, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj);
    return -2;
}

// conv3x3_tiled_dgrad_bn with the d-filter convolution of the same layer in the same kernel (see WgradFused);
// dx is not stored.  Returns -2 for shapes the fused form does not cover (then the two-kernel form applies).
int conv3x3_tiled_dgrad_bn_wgrad(hipStream_t s, const float* dz, const float* xc, const float* stats, const float* gamma,
                                  const float* totals, const float* in_records, int parts, float* dgamma, float* dbeta,
                                  const float* w, const float* add, float* out,
                                  const float* xc_post, const float* stats_post, float* records,
                                  const float* x_in, float* partial, const float* red_partial, float* red_dw, int red_E,
                                  int red_chunks, int N, int HW, int C) {
    if (!totals && !records_inline(parts, C)) return -1;
    BwdBn bwd;
    bwd.xc = xc; bwd.stats = stats; bwd.gamma = gamma; bwd.totals = totals; bwd.dx_out = nullptr;
    bwd.records = in_records; bwd.parts = parts; bwd.dgamma = dgamma; bwd.dbeta = dbeta;
    bwd.inv_m = 1.0f / (float)((long)N * HW * HW);
    PostBn post;
    post.mask_src = x_in; post.xc = xc_post; post.stats = stats_post; post.records = records;
    jobs::ReduceJob rj = jobs::ReduceJob();
    if (red_partial) {
        rj.partial = red_partial; rj.dw = red_dw; rj.E = red_E; rj.chunks = red_chunks;
        const int groups = jobs::reduce_groups(red_E, red_chunks);
        rj.blocks = groups < 288 ? groups : 288;
    }
    WgradFused wg;
    wg.x_in = x_in; wg.partial = partial;
    if (C == 16 && HW == 32) return launch<16, 32, 8, 1, true, 3, true, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj, wg);
    if (C == 32 && HW == 16) return launch<32, 16, 8, 1, true, 3, true, true>(s, dz, w, add, out, nullptr, N, PreBn(), post, bwd, rj, wg);
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
