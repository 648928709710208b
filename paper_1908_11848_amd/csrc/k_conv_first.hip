// First layer of the AlexNet-style networks, 5x5 (pad 2), 3 -> 64 channels on 32x32 images, with the 3x3 / stride 2 max-pool
// behind it, fp32 arithmetic on the bf16 matrix cores (split.hpp): forward with bias, ReLU and pooling in one pass; gradient
// w.r.t. filter and bias from the pooled gradient, without the 32x32x64 gradient ever existing in memory.
//
// What the layer cannot do without is the images and its pooled output (1.6 and 9.2 MB at batch 128); its products are 1.3 GFLOP.  The
// activations in front of the pooling (33.5 MB, most of what the forward kernel writes) are read by no kernel of a training step: they are
// stored for callers of dsspk_conv_first_pool_fwd and dssp_workspace_tensor, who check ReLU decisions on them.  Both
// directions use the image rows a band of output rows touches, laid out as patches: T[row][pixel][16] holds the 15
// neighbouring values (5 pixels x 3 channels, contiguous in memory) that a filter row meets at that pixel, and a zero, as
// three bf16 terms.  The reduction over a filter row is then 16 wide, and both operands of both directions are plain 8-byte
// or transposing LDS reads.
//
// Measured alone, batch 37 / 128 / 512: forward and pooling 10.9 / 16.3 / 55.8 us (as implicit GEMM on the fp32 matrix cores and a
// pooling kernel 17.8 / 37.0 / 122), gradients with their reduction 14.3 / 22.4 / 53.1 us (pooling backward, d-filter and column
// sums as kernels of their own 49 / 78 / 246).  Forward at batch 128 writes 41 MB: 2.6 TB/s; the rest is the patches'
// construction, then 4 us of matrix instructions, one after the other within a workgroup (two fit a compute unit).
#include "jobs.hpp"
#include "mma.hpp"
#include "split.hpp"
#include "conv_split_layers.hpp"
#include "../../include/dssp_kernels.h"

namespace {

constexpr int THREADS = 256;
constexpr int HW = 32, CI = 3, CO = 64, F = 5, PAD = 2, ROWF = F * CI;       // ROWF: values of a filter row at one pixel
constexpr int PW = 15;                                                      // pooled grid
constexpr int R = 8, BANDS = HW / R;                                        // output rows of a workgroup
constexpr int TPITCH = 3 * 32 + 8, TPLANE = 32;                             // bytes of a pixel of T, of one of its planes
constexpr int E = F * ROWF * CO;                                            // filter elements

// T rows for image rows h0 .. h0 + ROWS - 1.  A task is four values of one pixel's patch row.
template <int ROWS>
__device__ __forceinline__ void build_patches(const float* __restrict__ x, int n, int h0, char* T, int tid) {
    constexpr int TASKS = ROWS * HW * 4, LOADS = (TASKS + THREADS - 1) / THREADS;
    const split::Buffer img = split::buffer(x + (long)n * HW * HW * CI, 4u * HW * HW * CI);
    float4 v[LOADS];
#pragma unroll
    for (int e = 0; e < LOADS; ++e) {
        const int idx = tid + e * THREADS, c = idx & 3, px = (idx >> 2) % HW, row = (idx >> 2) / HW;
        const int h = h0 + row, at = CI * (px - PAD) + 4 * c;
        float f[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = (unsigned)h < (unsigned)HW && (unsigned)(at + i) < (unsigned)(HW * CI) && 4 * c + i < ROWF;
            f[i] = __uint_as_float(split::load1(img, in ? 4u * (unsigned)(h * HW * CI + at + i) : split::OUTSIDE));
        }
        v[e] = make_float4(f[0], f[1], f[2], f[3]);
    }
#pragma unroll
    for (int e = 0; e < LOADS; ++e) {
        const int idx = tid + e * THREADS;
        if (idx >= TASKS) break;
        uint2 pl[split::PLANES];
        split::split4(split::scaled(v[e]), pl);
#pragma unroll
        for (int p = 0; p < split::PLANES; ++p) *reinterpret_cast<uint2*>(T + (idx >> 2) * TPITCH + p * TPLANE + 8 * (idx & 3)) = pl[p];
    }
}

// ---------------------------------------------------------------------------------------------
// forward.  A workgroup owns 8 output rows of one image and the pooling windows that start in them, for which it computes the
// ninth row too; wavefront w owns output channels 16 w .. 16 w + 15, its filter operands in registers, and walks down the
// T rows: an operand serves the (up to five) output rows it meets at once.  A finished row goes to memory and to a three-row
// LDS ring of the wavefront's own, from which it takes the maxima.
constexpr int ROWS_F = R + 1;                                               // computed rows
constexpr int RING_PITCH = 16 * 4 + 16, RING_ROW = HW * RING_PITCH, RING = 3 * RING_ROW;
constexpr int FWD_LDS = (ROWS_F + F - 1) * HW * TPITCH + 4 * RING;

template <class... Job>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2))) void conv_first_kernel(
    const float* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias, float* __restrict__ a,
    float4* __restrict__ pooled, uchar4* __restrict__ arg, int own_blocks, Job... job) {
    if constexpr (sizeof...(Job) > 0)
        if ((int)blockIdx.x >= own_blocks) return (..., convert_filters(job, blockIdx.x - own_blocks));
    extern __shared__ __attribute__((aligned(16))) char lds_bytes[];
    char* T = lds_bytes;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, q = lane >> 4;
    char* ring = lds_bytes + (ROWS_F + F - 1) * HW * TPITCH + wave * RING;
    const int tile = xcd_tile(blockIdx.x, own_blocks), n = tile / BANDS, band = tile % BANDS, r0 = band * R;

    float4 fr[F][1];
#pragma unroll
    for (int k = 0; k < F; ++k) {
        const float* wp = w + (k * ROWF + 4 * q) * CO + 16 * wave + l16;
        fr[k][0] = make_float4(wp[0], wp[CO], wp[2 * CO], wp[q < 3 ? 3 * CO : 2 * CO]);         // all of them in flight together
    }
    const int co = 16 * wave + 4 * q;
    const float4 b = *reinterpret_cast<const float4*>(bias + co);
    build_patches<ROWS_F + F - 1>(x, n, r0 - PAD, T, tid);
    split::Filt<16> filt[F];
#pragma unroll
    for (int k = 0; k < F; ++k) {
        if (q == 3) fr[k][0].w = 0.f;               // a filter row has 15 values
        fr[k][0] = split::scaled(fr[k][0]);
        filt[k] = split::filter_operand<16>(fr[k]);
    }
    __syncthreads();

    floatx4 hi[ROWS_F][2], lo[ROWS_F][2];
#pragma unroll
    for (int r = 0; r < ROWS_F; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h) hi[r][h] = lo[r][h] = floatx4{0.f, 0.f, 0.f, 0.f};
    const char* base = T + l16 * TPITCH + 8 * q;
    split::Pix<16> op[2][2];
    auto load = [&](int t) {
#pragma unroll
        for (int h = 0; h < 2; ++h) op[t & 1][h] = split::pixel_operand<16, TPLANE>(base + (t * HW + 16 * h) * TPITCH);
    };
    const int rows = band == BANDS - 1 ? R : ROWS_F;
    auto store = [&](int r, int h, const floatx4& sum, float factor) {
        const float4 v = make_float4(fmaxf(fmaf(sum[0], factor, b.x), 0.f), fmaxf(fmaf(sum[1], factor, b.y), 0.f),
                                     fmaxf(fmaf(sum[2], factor, b.z), 0.f), fmaxf(fmaf(sum[3], factor, b.w), 0.f));
        const int px = 16 * h + l16;
        if (r < R) *reinterpret_cast<float4*>(a + (((long)n * HW + r0 + r) * HW + px) * CO + co) = v;
        *reinterpret_cast<float4*>(ring + r % 3 * RING_ROW + px * RING_PITCH + 16 * q) = v;
    };
    auto pool = [&](int r) {
        if (r < 2 || r % 2) return;
        // window row (r0 + r) / 2 - 1: the ring's three rows.  Lane (l16, q): window column l16 (15 of them), channels co ..
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (l16 < PW) {
            float4 best = make_float4(0.f, 0.f, 0.f, 0.f);
            uchar4 bi = make_uchar4(0, 0, 0, 0);
#pragma unroll
            for (int k = 0; k < 9; ++k) {        // first maximum in scan order, per channel
                const float4 v = *reinterpret_cast<const float4*>(ring + (r - 2 + k / 3) % 3 * RING_ROW + (2 * l16 + k % 3) * RING_PITCH + 16 * q);
                if (k == 0) { best = v; continue; }
                if (v.x > best.x) { best.x = v.x; bi.x = (unsigned char)k; }
                if (v.y > best.y) { best.y = v.y; bi.y = (unsigned char)k; }
                if (v.z > best.z) { best.z = v.z; bi.z = (unsigned char)k; }
                if (v.w > best.w) { best.w = v.w; bi.w = (unsigned char)k; }
            }
            const long o = (((long)n * PW + (r0 + r) / 2 - 1) * PW + l16) * (CO / 4) + co / 4;
            pooled[o] = best;
            arg[o] = bi;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    float bad = 0.f;
    load(0);
#pragma unroll
    for (int t = 0; t < ROWS_F + F - 1; ++t) {
        if (t + 1 < ROWS_F + F - 1) load(t + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int k = 0; k < F; ++k) {
                const int r = t - k;
                if (r < 0 || r >= ROWS_F) continue;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    floatx4& to = p < 2 ? lo[r][h] : hi[r][h];
                    to = split::product<16>(p, filt[k], op[t & 1][h], to);
                }
            }
        __builtin_amdgcn_sched_barrier(0);
        const int r = t - (F - 1);
        if (r < 0 || r >= rows) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const floatx4 sum = hi[r][h] + lo[r][h];
            bad = split::spoil(sum, bad);
            store(r, h, sum, split::UNSCALE);
        }
        pool(r);
    }
    if (!split::spoiled(bad)) return;
    // Some sum is beyond the range of the scaled terms: the wavefront's rows once more, those with such a sum from the operands in memory
    // (a lane with four of a filter row's values at its pixel, as in the patches), the others as above, so that a row that two
    // bands compute is the same in both.
#pragma unroll 1
    for (int r = 0; r < rows; ++r) {
        floatx4 sum[2], small[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) sum[h] = small[h] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < F; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const split::Pix<16> o = split::pixel_operand<16, TPLANE>(base + ((r + k) * HW + 16 * h) * TPITCH);
                small[h] = split::product<16>(0, filt[k], o, small[h]);
                small[h] = split::product<16>(1, filt[k], o, small[h]);
                sum[h] = split::product<16>(2, filt[k], o, sum[h]);
            }
        mma::drain();
#pragma unroll
        for (int h = 0; h < 2; ++h) sum[h] += small[h];
        float factor = split::UNSCALE;
        if (split::spoiled(split::spoil(sum[1], split::spoil(sum[0], 0.f)))) {
            factor = 1.f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                sum[h] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int k = 0; k < F; ++k) {
                    const int row = r0 + r + k - PAD, at = CI * (16 * h + l16 - PAD) + 4 * q;
                    float wv[4], xv[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const bool e = 4 * q + i < ROWF;
                        wv[i] = e ? w[(k * ROWF + 4 * q + i) * CO + 16 * wave + l16] : 0.f;
                        xv[i] = e && (unsigned)row < (unsigned)HW && (unsigned)(at + i) < (unsigned)(HW * CI) ? x[((long)n * HW + row) * HW * CI + at + i] : 0.f;
                    }
                    sum[h] = split::product32(wv, xv, sum[h]);
                }
            }
            mma::drain();
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) store(r, h, sum[h], factor);
        pool(r);
    }
}

// ---------------------------------------------------------------------------------------------
// d-filter and bias gradient, stage 1 of 2.  A workgroup walks its chunk's bands of 8 rows; per two image rows every thread
// takes one 2x2 block of pixels and four channels, fetches the four pooling windows that can route a gradient there
// (dy where the pooled output is positive, which is the ReLU's mask at the chosen pixel), adds them in window order and leaves
// the block as three bf16 terms in LDS.  dw[kh][e][co] += T[row + kh][pixel][e] d[row][pixel][co], pixels as reduction index,
// an image row to an MFMA, both operands by transposing reads; wavefront w: output channels 16 w .., all filter rows.
// Output: partial[chunk][E + 64 bias sums].
constexpr int DPITCH = 3 * 2 * CO + 16, DPLANE = 2 * CO;
constexpr int TBYTES = (R + F - 1) * HW * TPITCH, WGRAD_LDS = TBYTES + 2 * HW * DPITCH;

__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2))) void conv_first_wgrad_kernel(
    const float* __restrict__ x, const float* __restrict__ dpool, const float* __restrict__ pooled, const uint8_t* __restrict__ arg,
    float* __restrict__ partial, int items, int per_chunk) {
    extern __shared__ __attribute__((aligned(16))) char lds_bytes[];
    char *T = lds_bytes, *D = lds_bytes + TBYTES;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, q = lane >> 4;
    const int i0 = blockIdx.x * per_chunk, i1 = min(items, i0 + per_chunk);
    constexpr int SUBS = R / 2;

    // this thread's block column and channels; its four windows (block row - 1 or 0, column - 1 or 0) of the next two rows
    const int bj = tid >> 4, c4 = tid & 15;
    float4 g[4], pv[4];
    unsigned ar[4];
    auto fetch = [&](int item, int s) {
        const int n = item / BANDS, bi = item % BANDS * SUBS + s;
        const long o = (long)n * PW * PW * CO;
        const split::Buffer db = split::buffer(dpool + o, 4u * PW * PW * CO), pb = split::buffer(pooled + o, 4u * PW * PW * CO),
                            ab = split::buffer(arg + o, 1u * PW * PW * CO);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = bi - 1 + (k >> 1), j = bj - 1 + (k & 1);
            const bool in = (unsigned)i < (unsigned)PW && (unsigned)j < (unsigned)PW;      // no window there: zero gradient
            const unsigned at = (unsigned)((i * PW + j) * CO + 4 * c4);
            g[k] = split::load4(db, in ? 4u * at : split::OUTSIDE);
            pv[k] = split::load4(pb, in ? 4u * at : split::OUTSIDE);
            ar[k] = split::load1(ab, in ? at : split::OUTSIDE);
        }
    };
    float4 sb = make_float4(0.f, 0.f, 0.f, 0.f);
    auto stage = [&]() {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            g[k].x = pv[k].x > 0.f ? g[k].x : 0.f; g[k].y = pv[k].y > 0.f ? g[k].y : 0.f;
            g[k].z = pv[k].z > 0.f ? g[k].z : 0.f; g[k].w = pv[k].w > 0.f ? g[k].w : 0.f;
        }
#pragma unroll
        for (int dr = 0; dr < 2; ++dr)
#pragma unroll
            for (int dc = 0; dc < 2; ++dc) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int wr = dr + 2 * (1 - (k >> 1)), wc = dc + 2 * (1 - (k & 1));      // the pixel's place in window k
                    if (wr > 2 || wc > 2) continue;
                    const unsigned want = 3 * wr + wc;
                    v.x += (ar[k] & 255u) == want ? g[k].x : 0.f;
                    v.y += (ar[k] >> 8 & 255u) == want ? g[k].y : 0.f;
                    v.z += (ar[k] >> 16 & 255u) == want ? g[k].z : 0.f;
                    v.w += ar[k] >> 24 == want ? g[k].w : 0.f;
                }
                sb.x += v.x; sb.y += v.y; sb.z += v.z; sb.w += v.w;
                uint2 pl[split::PLANES];
                split::split4(split::scaled(v), pl);
#pragma unroll
                for (int p = 0; p < split::PLANES; ++p)
                    *reinterpret_cast<uint2*>(D + (dr * HW + 2 * bj + dc) * DPITCH + p * DPLANE + 8 * c4) = pl[p];
            }
    };
    // transposing reads: this lane names pixels 8 q + 4 h + l16 / 4 of an image row
    const char *ta[2], *da[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int p = 8 * q + 4 * h + (l16 >> 2);
        ta[h] = T + p * TPITCH + 8 * (l16 & 3);
        da[h] = D + p * DPITCH + 8 * (l16 & 3) + 32 * wave;
    }
    floatx4 hi[F], lo[F];
#pragma unroll
    for (int k = 0; k < F; ++k) hi[k] = lo[k] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (i0 < i1) fetch(i0, 0);
    for (int item = i0; item < i1; ++item) {
        build_patches<R + F - 1>(x, item / BANDS, item % BANDS * R - PAD, T, tid);
        uint4 t[F + 1][split::PLANES], d[2][split::PLANES];         // T rows 2 s .. 2 s + 5, row r in slot r mod 6
#pragma unroll
        for (int s = 0; s < SUBS; ++s) {
            stage();
            __syncthreads();
            if (s + 1 < SUBS) fetch(item, s + 1);
            else fetch(min(item + 1, i1 - 1), 0);                   // past the chunk's end: never used
#pragma unroll
            for (int j = 0; j < 2; ++j) split::transposed_operand<DPLANE>(d[j], da[0] + j * HW * DPITCH, da[1] + j * HW * DPITCH);
#pragma unroll
            for (int r = s ? 2 * s + F - 1 : 0; r < 2 * s + F + 1; ++r)
                split::transposed_operand<TPLANE>(t[r % (F + 1)], ta[0] + r * HW * TPITCH, ta[1] + r * HW * TPITCH);
            constexpr int PD[6] = {0, 2, 1, 0, 1, 0}, PT[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int p = 0; p < 6; ++p)
#pragma unroll
                    for (int k = 0; k < F; ++k) {
                        floatx4& to = p < 5 ? lo[k] : hi[k];
                        to = split::mfma(d[j][PD[p]], t[(2 * s + j + k) % (F + 1)][PT[p]], to);
                    }
            __syncthreads();                                        // both tiles are consumed
        }
    }
    mma::drain();
    float bad = 0.f;
#pragma unroll
    for (int k = 0; k < F; ++k) {
        hi[k] += lo[k];
        bad = split::spoil(hi[k], bad);
    }
    if (split::spoiled(bad)) {      // beyond the range of the scaled terms: this wavefront's sums from the operands in memory, four pixels a step
#pragma unroll
        for (int k = 0; k < F; ++k) hi[k] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int px = i0 * R * HW + q; px < i1 * R * HW; px += 4) {
            const int n = px / (HW * HW), h = px / HW % HW, c = px % HW, co = 16 * wave + l16, at = CI * (c - PAD) + l16;
            float d = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {       // the (up to) four windows of the pixel, in the order of stage()
                const int i = h / 2 - 1 + (k >> 1), j = c / 2 - 1 + (k & 1), wr = h - 2 * i, wc = c - 2 * j;
                if ((unsigned)i >= (unsigned)PW || (unsigned)j >= (unsigned)PW || wr > 2 || wc > 2) continue;
                const long o = (((long)n * PW + i) * PW + j) * CO + co;
                if (arg[o] == 3 * wr + wc && pooled[o] > 0.f) d += dpool[o];
            }
            const float dv[1] = {d};
#pragma unroll
            for (int k = 0; k < F; ++k) {
                const int row = h + k - PAD;
                const bool in = l16 < ROWF && (unsigned)row < (unsigned)HW && (unsigned)at < (unsigned)(HW * CI);
                const float xv[1] = {in ? x[((long)n * HW + row) * HW * CI + at] : 0.f};
                hi[k] = split::product32(dv, xv, hi[k]);
            }
        }
        mma::drain();
    } else {
#pragma unroll
        for (int k = 0; k < F; ++k) hi[k] *= split::UNSCALE;
    }
    float* out = partial + (long)blockIdx.x * (E + CO);
    if (l16 < ROWF)
#pragma unroll
        for (int k = 0; k < F; ++k) *reinterpret_cast<floatx4*>(out + (k * ROWF + l16) * CO + 16 * wave + 4 * q) = hi[k];
    float4* red = reinterpret_cast<float4*>(lds_bytes);             // bias: the 16 threads of one channel group, in order
    red[tid] = sb;
    __syncthreads();
    if (tid < 16) {
        float4 s = red[tid];
        for (int j = 1; j < THREADS / 16; ++j) { const float4 v = red[tid + 16 * j]; s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w; }
        *reinterpret_cast<float4*>(out + E + 4 * tid) = s;
    }
}

// Chunks: two workgroups fit a compute unit, so up to 512 run at once; beyond that a workgroup takes several bands.
int bands_per_chunk(int N) { return ceil_div((long)N * BANDS, 512); }

template <class K>
int allow_lds(K kern, int bytes, bool& done) {           // raise the dynamic-LDS limit once per kernel
    if (done) return 0;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) return -1;
    done = true;
    return 0;
}

}  // namespace

__global__ __launch_bounds__(SplitFilterJob::THREADS) void convert_filters_kernel(SplitFilterJob job) { convert_filters(job, blockIdx.x); }

template <class... Job>
static int launch_fwd(hipStream_t s, const float* x, const float* w, const float* bias, float* a, float* pooled, uint8_t* arg, int N, int more_blocks,
                      const Job&... job) {
    if (!x || !w || !bias || !a || !pooled || !arg || N < 1 || (long)N * HW * HW >= 1L << 31) return -1;
    static bool done = false;
    if (allow_lds(conv_first_kernel<Job...>, FWD_LDS, done)) return -1;
    hipLaunchKernelGGL((conv_first_kernel<Job...>), dim3(N * BANDS + more_blocks), dim3(THREADS), FWD_LDS, s, x, w, bias, a, reinterpret_cast<float4*>(pooled),
                       reinterpret_cast<uchar4*>(arg), N * BANDS, job...);
    return DSSPK_LAUNCH_RC();
}

int conv_first_pool_fwd(hipStream_t s, const float* x, const float* w, const float* bias, float* a, float* pooled, uint8_t* arg, int N, SplitFilterJob job) {
    // Not where the job alone would begin a second round of workgroups, two to a compute unit.  A round of pushes, two 5x5 layers, conversion by
    // a launch of its own / carried, us: batch 128, four workers 631 / 637 and 633 / 649, 95 492 / 490, 512, two workers 1102 / 1088; three
    // convolutions: batch 37 408 / 390, 140 769 / 760.
    constexpr int ROUND = 2 * 256;
    const int own = N * BANDS;
    if (own > ROUND || own + job.blocks() <= ROUND) return launch_fwd(s, x, w, bias, a, pooled, arg, N, job.blocks(), job);
    if (const int rc = launch_fwd(s, x, w, bias, a, pooled, arg, N, 0)) return rc;
    hipLaunchKernelGGL(convert_filters_kernel, dim3(job.blocks()), dim3(SplitFilterJob::THREADS), 0, s, job);
    return DSSPK_LAUNCH_RC();
}

extern "C" int dsspk_conv_first_pool_fwd(void* stream, const float* x, const float* w, const float* bias, float* a, float* pooled,
                                         uint8_t* arg, int N) {
    return launch_fwd((hipStream_t)stream, x, w, bias, a, pooled, arg, N, 0);
}

extern "C" size_t dsspk_conv_first_scratch_floats(int N) {
    return N < 1 ? 0 : (size_t)ceil_div((long)N * BANDS, bands_per_chunk(N)) * (E + CO);
}

int conv_first_pool_bwd_weight_parts(hipStream_t stream, const float* x, const float* dpooled, const float* pooled, const uint8_t* arg, float* dw,
                                     float* scratch, int N, jobs::Partials* waiting) {
    if (!x || !dpooled || !pooled || !arg || !dw || !scratch || N < 1 || (long)N * HW * HW >= 1L << 31) return -1;
    static bool done = false;
    if (allow_lds(conv_first_wgrad_kernel, WGRAD_LDS, done)) return -1;
    const int per = bands_per_chunk(N), chunks = ceil_div((long)N * BANDS, per);
    hipLaunchKernelGGL(conv_first_wgrad_kernel, dim3(chunks), dim3(THREADS), WGRAD_LDS, stream, x, dpooled, pooled, arg, scratch,
                       N * BANDS, per);
    *waiting = {scratch, dw, E + CO, chunks, false};
    return DSSPK_LAUNCH_RC();
}

extern "C" int dsspk_conv_first_pool_bwd_weight(void* stream, const float* x, const float* dpooled, const float* pooled, const uint8_t* arg,
                                                float* dw, float* scratch, int N) {
    jobs::Partials p;
    if (const int rc = conv_first_pool_bwd_weight_parts((hipStream_t)stream, x, dpooled, pooled, arg, dw, scratch, N, &p)) return rc;
    return dsspk_wgrad_reduce(stream, p.partial, p.dw, p.E, p.chunks);
}
