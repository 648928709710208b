// 3x3, stride 1, pad 1 convolutions with Cin = Cout = C (the 106 inner convolutions of
// ResNet-110): forward and gradient w.r.t. the input as ONE kernel.
//
// A workgroup owns a band of R output rows of one image (or all of them) and CN of the C output channels, and has four or eight
// wavefronts of four pixel tiles each, or four wavefronts of two (k_conv3x3.hip, k_conv3x3_large.hip, k_conv3x3_small.hip).  It loads the
// (R+2) x (HW+2) x C input halo tile (zero borders) into LDS once; everything else is served from LDS, so every input element is read from
// memory once per band instead of nine times.  The filter never passes through LDS: a wavefront owns ONE tile of 16 output channels and holds
// one column of that tile's filter (three taps) in registers; a row of the next column is fetched while the products still work with the present
// one.  In a network's step the filter comes already split (conv3x3_filter.hpp), with two pixel tiles two columns are held, and what is not needed
// at once is fetched between the products.  Callers of single layers have the filter split here; with two pixel tiles all three columns and
// everything else are then fetched up front.  LDS holds the halo tile and a little for the sums: 36 to 45 KB with four wavefronts, 46 to 82 KB with
// eight, 22 to 45 KB with two pixel tiles (the last stage's d-filter beside its d-input: 61).  Registers are at most 128 with eight wavefronts, and
// what fits a compute unit of LDS and registers overlaps: one workgroup's transfers run beside another's products.
//
// What bounds them (110 layers, batch 128, four streams, measured where a push took 1.82 ms): registers and LDS admit 16 wavefronts to a compute unit and each
// fetches, multiplies and stores one after the other.  Without the products a push takes 1.27 ms (its bytes at copy rate: 1.0), without
// the fused d-filter 1.60, without the epilogue's loads 1.74.  Therefore: no spilled register (with one to 17 of them per kernel
// 1.86 ms), addresses as 32-bit offsets from a uniform base, and nothing held across the product loop that the thread index gives.
//
// The arithmetic is fp32 on the bf16 matrix cores (split.hpp): the loader leaves every element in LDS as three bf16 terms
// (each converted once, not once per tap), the filter values come split or are split in registers while the input is on its way, and
// six of the nine products are taken.  The matrix-core tile is 16 output channels (rows) x 16 pixels (columns); a wavefront owns
// one channel tile and four pixel tiles that lie below each other, so a pixel operand fetched for one filter row serves
// the tiles above it too, and a lane ends up with four consecutive channels of a pixel (16-byte loads and stores in the
// epilogue).
//
// Gradient w.r.t. the input of such a convolution is the same operation on dy with the filter
// taps reversed and its two channel indices swapped; only the filter fetch differs.
#pragma once
#include "mma.hpp"
#include "split.hpp"
#include "bn_merge.hpp"
#include "jobs.hpp"
#include "conv3x3_filter.hpp"

namespace {

// Records of the tensor in front that a thread of its consumer fetches at most
template <int C, int WAVES, int NT> constexpr int max_records() { return NT == 2 || (WAVES == 8 && C == 64) ? 16 : 8; }

template <int C, int HW, int R, int NSPLIT, int WAVES>
struct Cfg {
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int CN = C / NSPLIT;          // output channels per workgroup
    static constexpr int PLANE = 2 * C;            // bytes between the three bf16 terms of a pixel in LDS
    // Pitch of a pixel: 16 bytes behind its terms (C = 16: 8; 64: 32, and 192 behind a row).  LDS has 64 banks, and a 16-byte read is served 16
    // lanes at a time, 0-3, 12-15 and 20-27 first (measured read by read): so a pixel operand takes twice the steps it could with 32 channels (32 bytes
    // would not leave room for two workgroups, and dealing the 16-byte parts of a plane by the column changed no time) and no more than it
    // must with 64 (16 bytes: three times; a push of 50 layers, batch 128, one worker 1639 -> 1634 us, 20 layers, batch 8 383.3 -> 382.4).
    static constexpr int PITCH = 3 * PLANE + (C == 16 ? 8 : C == 32 ? 16 : 32);
    static constexpr int TW = HW + 2;              // halo tile width
    static constexpr int ROW = TW * PITCH + (C == 64 ? 192 : 0);       // bytes of a tile row
    static constexpr int XB = (R + 2) * ROW;
    static constexpr int WAVES_N = CN / 16;        // wavefronts side by side over the output channels
    static constexpr int WAVES_M = WAVES / WAVES_N;    // ... and over the pixels or, in the last stage, the input channels
    // A wavefront works on NT (four or two) pixel tiles, each one (HW >= 16) or two (HW = 8) image rows below the one before.
    static constexpr int TROWS = HW >= 16 ? 1 : 2;
    static constexpr int TX = HW >= 16 ? HW / 16 : 1;          // tiles side by side
    static constexpr int KS = C == 64 ? 2 : 1;     // wavefronts that share pixels and split the input channels; they swap
                                                   // halves of their sums through LDS and each finishes its half
    static constexpr int WPX = WAVES_M / KS;                   // wavefronts over the band's pixels
    static constexpr int NT = R * TX / (TROWS * WPX);
    static constexpr int WM = NT / KS;             // pixel tiles a wavefront finishes
    // Two tiles: the products of a filter column are too few to hide the fetch of the next one, and registers are not what counts
    // where the tiles are that small: all three columns are fetched up front (where the kernel splits the filter; see SPREAD).
    static constexpr int COLUMNS = NT == 4 ? 1 : 3;
    // ... and so is everything else the workgroup reads: one latency instead of three or four in a row (figures before the filters were converted
    // ahead).  A push of the 20-layer network, one
    // worker, without / with it, us: batch 1 440 / 434, 8 470 / 466, 16 485 / 481; four workers, a round: 830 / 820, 895 / 881, 920 / 900.
    static constexpr bool EARLY = NT == 2;
    static constexpr int SC = WAVES_M * CN;        // floats: per-wavefront column sums (batch-norm records, one component)
    static constexpr int SS = 2 * SC;
    static constexpr int PS = 5 * C;               // floats: per-channel vectors of the loader
    static constexpr int PX = 4 * C;               // ... and of the fused d-filter's x tile
    static constexpr size_t LDS_BYTES = XB + (size_t)(SS + PS) * sizeof(float);
    static constexpr size_t LDS_X = LDS_BYTES + PX * sizeof(float);        // with a fused d-filter
    // fused d-filter: the x halo tile takes the place of the first one.  A wavefront owns one 16x16 tile of (ci, co) and RUNS of the
    // band's runs of 32 pixels; RSPLIT wavefronts share a tile and their sums meet in LDS: C = 16 all nine taps at the end, in the
    // tile's place; C = 32 one filter column after the other, behind everything else.
    static constexpr int DTILES = C == 16 ? 1 : 4, RSPLIT = WAVES / DTILES, RUNS = R * HW / 32 / RSPLIT;
    static constexpr size_t RED = C == 16 ? (size_t)WAVES * 9 * C * C * sizeof(float) : 0;
    static constexpr size_t COLUMN = C == 32 && RSPLIT == 2 ? (size_t)DTILES * 3 * 256 * sizeof(float) : 0;
    // C = 64 (the output channels in four parts): the x tile, 16 channels of it, has a place of its own, and so has what wavefronts exchange.
    static constexpr int X2PLANE = 32, X2PITCH = 3 * X2PLANE + 8, X2 = (R + 2) * TW * X2PITCH;
    static constexpr size_t OWN_X = C == 64 ? X2 + (size_t)WAVES * WM * 64 * 16 : 0;
    // (RED takes everything's place)
    static constexpr size_t TWO = 80 * 1024;       // bytes of which a compute unit holds two
    static constexpr size_t WG_BYTES = LDS_X + COLUMN + OWN_X, LDS_BYTES_WG = WG_BYTES > RED ? WG_BYTES : RED;
    static_assert(WPX * KS == WAVES_M && (NT == 4 || NT == 2) && NT * TROWS * WPX == R * TX && (C == 16 || C == 32 * KS), "roles of the wavefronts");
    static_assert(WG_BYTES <= TWO && SS >= WAVES, "two workgroups to a compute unit");
    static_assert(XB % 16 == 0 && WAVES * 2 * 64 * 16 <= XB, "alignment; room for the exchange");
    // the loader: rows inside the image (or halo rows of a band), columns inside the image; what remains of the tile is zero
    static constexpr bool WHOLE = R == HW;
    static constexpr int ROWS = WHOLE ? R : R + 2, ROW0 = WHOLE ? 1 : 0;
    static constexpr int V = C / 4;                // 16-byte vectors of a pixel
    static constexpr int NL = (ROWS * HW * V + THREADS - 1) / THREADS;
    static constexpr int ZERO_UNIT = PITCH % 16 == 0 ? 16 : 8, ZERO_UNITS = 3 * PLANE / ZERO_UNIT;       // of a border pixel
    static constexpr int ZERO = (2 * (R + 2) + (WHOLE ? 2 * HW : 0)) * ZERO_UNITS;
    // records of the tensor in front: each thread fetches at most this many
    static constexpr int RECORDS = max_records<C, WAVES, NT>();
};

// Normalisation applied to the input while it is loaded (PRE != 0): the kernel then computes
//   a = ReLU(gamma * (src - mean) * invstd + beta (+ shortcut))   and   dst = conv(a),
// i.e. the batch norm + ReLU that separates two convolutions never runs as a pass of its own.
// mean / invstd come from the statistics records of src, merged by a small kernel launched just before or, if they are few
// (records_inline), by every workgroup itself; they are also what the backward pass needs.  The workgroups write `a` (their own rows).
// What a kernel is handed of it stands in the base; the rest are arguments of their own (conv3x3_kernel), which this description of a launch holds for
// the host alone.
struct PreArgs {
    long M, rows;              // of src (= N * HW * HW); of a record
    float eps;
    float* act_out;            // a
    float* stats_out;          // mean[C], invstd[C]
};
struct PreBn : PreArgs {
    const float* records;      // statistics records of src
    int parts;                 // how many
    const float* gamma;
    const float* beta;
    const float* shortcut;     // PRE == 2: added before the ReLU, same shape as src ...
    bool half;                 // ... or (C > 16) twice as high and wide with half the channels: every second pixel of it, zero beyond its channels
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
    const float *gamma, *beta; // of the batch norm (REPEAT)
};

// Batch-norm backward applied to the input while it is loaded (PRE == 3, d-input convolutions): src is dz, the
// masked gradient at the batch norm's output, and the convolution runs on
//   dx = gamma * invstd * (dz - sum(dz) / M - xhat * sum(dz * xhat) / M),   xhat = (xc - mean) * invstd,
// the gradient w.r.t. the batch norm's input xc; the workgroups also write dx (their own rows) for the
// d-filter kernel.  The two sums come from the records of the epilogue that produced dz: added up before (TotalsJob) or, if
// they are few, by every workgroup itself.
struct BwdArgs {
    const float* totals;       // sum dz [C], sum dz * xhat [C]; null: add up the records
    float *dgamma, *dbeta;     // with records: sum dz * xhat and sum dz, stored by the first workgroup
    float inv_m;               // 1 / (N * HW * HW)
    float* dx_out;
};
struct BwdBn : BwdArgs {
    const float* xc;           // the batch norm's input
    const float* stats;        // its mean[C], invstd[C]
    const float* gamma;
    const float* records;      // [parts][C][2]
    int parts;
};

// Gradient w.r.t. the filter in the same kernel (WG, only with PRE == 3; a workgroup has all output channels of the layer in its tile): the
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
// Wavefronts per SIMD the register allocation aims at: with eight wavefronts to a workgroup two of them per compute unit need four; with four
// to a workgroup the fourth brings nothing (a round of eight workers on four streams, three / four, us: 110 layers, batch 64 12390 / 12460, 50
// layers, batch 33 5760 / 5800).
// Two pixel tiles to a wavefront: no second workgroup waits for room on the compute unit.
template <int C, int WAVES, bool WG, int NT>
constexpr int min_waves() { return NT == 2 ? 2 : WAVES == 8 || (C == 16 && !WG) ? 4 : 3; }

// Sum over the 16 lanes of a quarter wavefront, in all of them.
__device__ __forceinline__ float sum16(float v) {
#define ROR(n) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + n, 0xf, 0xf, true))
    v += ROR(8); v += ROR(4); v += ROR(2); v += ROR(1);
#undef ROR
    return v;
}
__device__ __forceinline__ float4 sum16(float4 v) { return make_float4(sum16(v.x), sum16(v.y), sum16(v.z), sum16(v.w)); }

// The most records of a tensor that every workgroup of its consumer merges itself.
template <int C, int WAVES, int NT = 4> constexpr int inline_records() { return 64 * WAVES * max_records<C, WAVES, NT>() / C; }

// Thread (channel tid % C, lane tid / C) holds records lane, lane + THREADS / C, ... of its channel, behind the last one zeros: the list is a
// buffer, so neither its end nor an address takes vector instructions (68 before: a push of the 50-layer network, batch 128, one worker 1719 ->
// 1698 us).  A load beyond the end still takes its turn: all sixteen without a condition, 20 layers, batch 8, 349 -> 363 us.
template <int C, int THREADS, int RECORDS>
__device__ __forceinline__ void load_records(float2 (&v)[RECORDS], const float* __restrict__ records, int parts, int tid) {
    constexpr int FEW = 4;          // at a time: where a list is short its loads would keep those behind them waiting
    const split::Buffer list = split::buffer(records, 8u * (unsigned)(parts * C));
#pragma unroll
    for (int u0 = 0; u0 < RECORDS; u0 += FEW) {
        if (RECORDS > 8 && u0 * (THREADS / C) >= parts) {
#pragma unroll
            for (int u = u0; u < u0 + FEW; ++u) v[u] = make_float2(0.f, 0.f);
            continue;
        }
#pragma unroll
        for (int u = u0; u < u0 + FEW; ++u) v[u] = split::load2(list, 8u * (unsigned)(tid + u * THREADS));
    }
}
// ... and how many of a channel's the lanes of wavefront w hold together
template <int C, int THREADS> __device__ __forceinline__ int records_of(int parts, int w) {
    constexpr int LANES = THREADS / C, PER = 64 / C;
    return parts / LANES * PER + min(max(parts % LANES - w * PER, 0), PER);
}
template <int C, int THREADS> __device__ __forceinline__ bool has_record(int u, int parts, int tid) { return tid / C + u * (THREADS / C) < parts; }

// Sum over the lanes of a wavefront that share a channel (thread: channel tid % C), in all of them.
template <int C> __device__ __forceinline__ float lanes_sum(float v) {
    if constexpr (C <= 32) {
        const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    }
    if constexpr (C <= 16) {
        const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    }
    return v;
}

// Statistics records are merged (Chan's formula) by each wavefront for itself, its lanes by swaps of their registers, and the wavefronts meet
// once; with the mean of all first and then the deviations from it they met twice.  A push of 50 layers, batch 128, one worker / four 1650 / 786 ->
// 1638 / 776 us, 20 layers, batch 8 385 -> 383.
// A wavefront's share of the statistics records (mean, sum of squared deviations; of nn rows each), for the channel of the lane: the sum of the means,
// their mean, and the sum of squared deviations of all its rows from that.
struct Share { float sum, mean, m2; };
template <int C, int THREADS, int RECORDS>
__device__ __forceinline__ Share merge_lanes(const float2 (&rec)[RECORDS], int parts, float nn, int tid) {
    constexpr int LANES = THREADS / C, PER = 64 / C;        // that share a channel: of the workgroup, of a wavefront
    // (nothing is added to a zero: the compiler would move that up to the load, and the tile's loads would wait for the records)
    float s_ = rec[0].x, m2 = rec[0].y, d2, mean;
#pragma unroll
    for (int u = 1; u < RECORDS; ++u) s_ += rec[u].x;
    s_ = lanes_sum<C>(s_);
    if (parts == RECORDS * LANES) {
        mean = s_ * (1.f / (RECORDS * PER));
        d2 = (rec[0].x - mean) * (rec[0].x - mean);
#pragma unroll
        for (int u = 1; u < RECORDS; ++u) {
            const float d = rec[u].x - mean;
            m2 += rec[u].y;
            d2 = fmaf(d, d, d2);
        }
    } else {
        const int count = records_of<C, THREADS>(parts, __builtin_amdgcn_readfirstlane(tid >> 6));
        mean = count ? s_ / (float)count : 0.f;
        d2 = 0.f;
        constexpr int FEW = RECORDS < 4 ? RECORDS : 4;
#pragma unroll
        for (int u0 = 0; u0 < RECORDS; u0 += FEW) {
            if (u0 * LANES >= parts) continue;
#pragma unroll
            for (int u = u0; u < u0 + FEW; ++u) {
                const float d = has_record<C, THREADS>(u, parts, tid) ? rec[u].x - mean : 0.f;
                if (u) m2 += rec[u].y;
                d2 = fmaf(d, d, d2);
            }
        }
    }
    return {s_, mean, lanes_sum<C>(fmaf(nn, d2, m2))};
}

// ... and of all WAVES shares (at red, C of each wavefront's): the channel's mean and its sum of squared deviations.  What the shares' means add to that sum
// is small beside it and would cost it a rounding of its own; added up in 64 bits everything has one together.  Error of invstd against float64,
// relative, 1 to 128 images: 4.1e-8 to 4.6e-8 with all deviations taken from the mean of all, 4.3e-8 to 4.8e-8 by shares in 32 bits, 3.9e-8 to 4.3e-8 so.
template <int C, int WAVES, int RECORDS>
__device__ __forceinline__ float2 merge_waves(const Share* red, int parts, float nn, int c) {
    constexpr int THREADS = 64 * WAVES, LANES = THREADS / C, PER = 64 / C;
    Share v[WAVES];
    double m2[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        v[w] = red[w * C + c];
        m2[w] = (double)v[w].m2;
    }
    float mean = v[0].sum, d2 = 0.f;
#pragma unroll
    for (int w = 1; w < WAVES; ++w) mean += v[w].sum;
    if (parts == RECORDS * LANES) {
        mean *= 1.f / (RECORDS * LANES);
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float d = v[w].mean - mean;
            d2 = fmaf(d, d, d2);
        }
        d2 *= RECORDS * PER;
    } else {
        mean /= (float)parts;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float d = v[w].mean - mean;
            d2 = fmaf((float)records_of<C, THREADS>(parts, w) * d, d, d2);
        }
    }
#pragma unroll
    for (int n = WAVES / 2; n >= 1; n /= 2)
#pragma unroll
        for (int w = 0; w < n; ++w) m2[w] = m2[2 * w] + m2[2 * w + 1];
    return make_float2(mean, (float)(m2[0] + (double)(nn * d2)));
}

// PL: the filter's operands are there already, see conv3x3_filter.hpp
// REPEAT (POST): mask_src is ReLU(BN(xc)) with nothing added, so the mask and the fused d-filter's x tile are worked out from xc again, by the
// forward pass's own operations (the same bits), and a tensor less is read: a sixth of such a layer's bytes.  Reading it / so, a round of pushes, us:
// batch 128, eight workers, 110 layers 16513 / 16322, 50 layers 7633 / 7509; 56 layers, batch 95, four 3216 / 3200; small batches the same.  (In the
// last stage's d-filter kernel, where it would be a fourth of 6 MB, it changed nothing and was left out.)
// Arguments: the first 14 words are in registers when a wavefront starts (-amdgpu-kernarg-preload-count), so what the first loads need comes first:
// records, their number (0: merged or added up before) with 2^16 for a shortcut of twice the size, src, what is normalised with it (beside: shortcut, or the batch
// norm's input), the filter, gamma and beta (or statistics and gamma).  Anything else is a load from memory that those would wait for: a push of 50
// layers, batch 128, one worker 1624 -> 1565 us, 20 layers, batch 8 382 -> 360 (with the arguments in their old order 1612 and 377).
template <int C, int HW, int R, int NSPLIT, int WAVES, bool TRANSPOSED, int PRE, bool POST, bool WG, bool PL, bool REPEAT>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(min_waves<C, WAVES, WG, Cfg<C, HW, R, NSPLIT, WAVES>::NT>()))) void conv3x3_kernel(
    const float* __restrict__ records, int list, int conv_blocks, const float* __restrict__ src, const float* __restrict__ beside, const uint4* __restrict__ planes,
    const float* __restrict__ norm_first, const float* __restrict__ norm_second, const float* __restrict__ wgt, const float* add, float* dst,
    float* __restrict__ bn_partial, PreArgs pre, PostBn post, BwdArgs bwd, jobs::ReduceJob rj, WgradFused wg) {
    using K = Cfg<C, HW, R, NSPLIT, WAVES>;
    constexpr int THREADS = K::THREADS, V = K::V, NL = K::NL;
    // Filter columns in registers.  With converted filters and two pixel tiles the next one's rows, and then what the epilogue reads and the
    // fused d-filter's x tile, are fetched between the products (SPREAD): in front of them the records and the tile wait behind some fifty other
    // loads a wavefront, each 16 cycles of the compute unit's address unit (batch 8, cycles until the records are summed: 5 to 7 thousand; it is
    // also 50 to 90 registers less).  All loads in front / so, a round of pushes, us: 20 layers, batch 8, four workers 678 / 652, batch 17, three
    // 580 / 577; 50 layers, batch 8, two 1143 / 1059; 110 layers, batch 3, eight 7677 / 7177.
    constexpr bool SPREAD = PL && K::EARLY;
    constexpr int COLUMNS = SPREAD ? 2 : K::COLUMNS;
    static_assert(!WG || (PRE == 3 && TRANSPOSED && (C == 64 ? NSPLIT == 4 && SPREAD : NSPLIT == 1)), "fused d-filter: d-input form");
    extern __shared__ __attribute__((aligned(16))) char lds_bytes[];
    char* lds = lds_bytes;
    if ((int)blockIdx.x >= conv_blocks) {           // workgroups behind the convolution's own carry the reduction job
        jobs::wgrad_reduce<THREADS>(rj, blockIdx.x - conv_blocks, reinterpret_cast<float*>(lds));
        __builtin_amdgcn_endpgm();
        __builtin_unreachable();
    }
    const int parts = list & 0xffff;                // 0: already merged, or added up
    const bool half = list >> 16;
    char* Xs = lds;
    float* Ss = reinterpret_cast<float*>(lds + K::XB);          // column sums
    float* Sh = Ss + K::SS;                                     // per-channel vectors of the loader
    const int tid = threadIdx.x;
    constexpr int BANDS = HW / R;
    const int tile = xcd_tile(blockIdx.x, conv_blocks);
    const int part = tile % NSPLIT;
    const int band = (tile / NSPLIT) % BANDS;
    const int n = tile / (NSPLIT * BANDS);
    const int r_base = band * R;                    // first output row of the band
    const long image_at = (long)n * HW * HW * C;
    const long band_at = image_at + (long)r_base * HW * C;
    // What a lane does follows from its thread index alone; behind the product loop it is worked out again, so that none of it takes
    // registers during the loop.
    struct Role { int lane, wave, l16, q, wave_n, wave_m, co_w, wpx, ks, row0, col; };
    auto role_of = [&](int t) {
        Role r;
        r.lane = t & 63; r.wave = t >> 6; r.l16 = r.lane & 15; r.q = r.lane >> 4;
        r.wave_n = r.wave % K::WAVES_N; r.wave_m = r.wave / K::WAVES_N;
        r.co_w = part * K::CN + 16 * r.wave_n;                  // first output channel of this wavefront
        r.wpx = r.wave_m / K::KS; r.ks = r.wave_m % K::KS;      // its pixels, its share of the input channels
        r.row0 = r.wpx / K::TX * K::NT * K::TROWS + (K::TROWS == 2 ? r.l16 >> 3 : 0);           // this lane's pixel in the first tile
        r.col = K::TROWS == 2 ? r.l16 & 7 : 16 * (r.wpx % K::TX) + r.l16;
        return r;
    };
    auto load4 = [](const float* base, unsigned off) { return *reinterpret_cast<const float4*>(base + off); };

    // ---- filter values of this lane, result channel co_w + l16 (row of the MFMA tile) and reduction channels k0 ..:
    //      forward : w[tap][k][co]           (C floats apart)
    //      d-input : w[8 - tap][co][k]       (16-byte loads, taps reversed)
    //      One filter column (three taps) at a time: the product loop walks the columns, and a row of the next one is
    //      fetched while the loop still works with that row of the present one.
    constexpr int FV = C == 16 ? 1 : 2;
    float4 fr[PL ? 1 : COLUMNS][3][FV];
    split::Filt<C> filt[PL ? COLUMNS : 1][3];
    unsigned filter_at;
    if constexpr (PL) {
        const Role r = role_of(tid);
        filter_at = ((C == 64 ? 4 * r.ks : 0) + r.co_w / 16) * filter3x3_quads(C) * 64 + r.lane;
    } else {
        const Role r = role_of(tid);
        const int k0 = C == 16 ? 4 * r.q : 32 * r.ks + 8 * r.q;
        filter_at = TRANSPOSED ? (r.co_w + r.l16) * C + k0 : k0 * C + r.co_w + r.l16;
    }
    auto load_filter = [&](int ky, int kx) {
        const int tap = 3 * ky + kx;
        if constexpr (PL) {
#pragma unroll
            for (int p = 0; p < filter3x3_quads(C); ++p)
                filt[kx % COLUMNS][ky].v[C == 16 ? 2 * p : p] = (planes + (tap * (filter3x3_operands(C) / 9) * filter3x3_quads(C) + p) * 64)[filter_at];
        } else {
#pragma unroll
            for (int e = 0; e < FV; ++e) {
                if constexpr (TRANSPOSED) {
                    fr[kx % COLUMNS][ky][e] = load4(wgt + (8 - tap) * C * C + 4 * e, filter_at);
                } else {
                    const float* wp = wgt + tap * C * C + 4 * e * C;
                    fr[kx % COLUMNS][ky][e] = make_float4((wp + 0 * C)[filter_at], (wp + 1 * C)[filter_at], (wp + 2 * C)[filter_at], (wp + 3 * C)[filter_at]);
                }
            }
        }
    };
    auto split_filter = [&](int ky, int kx) {
        if constexpr (!PL) {
            float4 (&f)[FV] = fr[kx % COLUMNS][ky];
#pragma unroll
            for (int e = 0; e < FV; ++e) f[e] = split::scaled(f[e]);
            filt[0][ky] = split::filter_operand<C>(f);
        }
    };
    auto first_columns = [&]() {
#pragma unroll
        for (int kx = 0; kx < (SPREAD ? 1 : COLUMNS); ++kx)
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) load_filter(ky, kx);
    };
    // What the loader needs of the batch norm (PRE 1, 2: of this thread's channels; 3: of channel tid), fetched with everything else: read where
    // it is used, behind the sums and once a vector of the tile, each vector waits for memory again.  A push of the 50-layer network, batch
    // 128, one worker / four, us: 1688 / 806, so 1669 / 795; with the vectors of the tile's channels read from LDS once, 1660 / 798.
    float4 norm_g = make_float4(0.f, 0.f, 0.f, 0.f), norm_b = norm_g;
    float norm_mean = 0.f, norm_is = 0.f, norm_gamma = 0.f;
    if constexpr (PRE == 1 || PRE == 2) {
        norm_g = *reinterpret_cast<const float4*>(norm_first + tid % V * 4);
        norm_b = *reinterpret_cast<const float4*>(norm_second + tid % V * 4);
    }
    if constexpr (PRE == 3)
        if (tid < C) { norm_mean = norm_first[tid]; norm_is = norm_first[C + tid]; norm_gamma = norm_second[tid]; }
    // The filter is new to every L2, and workgroups that keep step with each other all wait for each of its rows in turn.  With eight wavefronts
    // the workgroups of an XCD therefore touch a line of it a thread, each its share, before they do anything else.  A push of 50 layers, batch 128,
    // one worker 1635 -> 1624 us, a round of eight workers 7024 -> 6952.  (Smaller workgroups: nothing, two such loads a thread cost as much.  The
    // epilogue's operands touched in the same way: 1660 -> 1688.)
    constexpr bool WARM = PL && WAVES == 8;
    unsigned warm = 0;
    if constexpr (WARM) {
        constexpr int LINES = (int)(filter3x3_uint4s(C) / 8);
        const int groups = conv_blocks / 8, share = groups ? (LINES + groups - 1) / groups : 0, at = blockIdx.x / 8 * share + tid;
        if (tid < share && at < LINES) warm = planes[8 * at].x;
    }
    float2 rec[PRE ? K::RECORDS : 1];
    if constexpr (PRE == 1 || PRE == 2)
        if (parts) load_records<C, THREADS>(rec, records, parts, tid);
    if constexpr (PRE == 3)
        if (parts) load_records<C, THREADS>(rec, records, parts, tid);
    if constexpr (!PL) first_columns();
    // ---- input halo tile, zero outside the image.  The raw loads are issued first; the first filter column is split while
    //      they are in flight.
    float4 val[NL], scv[PRE >= 2 ? NL : 1];
    // Vectors of this thread: one of the tile's first rows and those RE, 2 RE, .. rows below it; one after the other in memory.
    constexpr int RE = THREADS / (V * HW);
    static_assert(RE * V * HW == THREADS && NL == (K::ROWS + RE - 1) / RE, "whole rows");
    const int pr0 = tid / (V * HW), c4 = tid % V * 4;
    const long tile_at = image_at + (r_base + K::ROW0 - 1) * HW * C;       // may lie in front of the image, where nothing is fetched
    char* tile_to = Xs + (pr0 + K::ROW0) * K::ROW + (tid / V % HW + 1) * K::PITCH + 2 * c4;
    constexpr int STEP = RE * HW * C, STEP_TO = RE * K::ROW;
    auto own = [&](int e) { return (e + 1) * RE <= K::ROWS || pr0 + e * RE < K::ROWS; };                            // a row of the tile
    auto inside = [&](int e) { return K::WHOLE || (own(e) && (unsigned)(r_base - 1 + pr0 + e * RE) < (unsigned)HW); };   // and of the image
    // Nothing up to here and none of these loads stands behind a branch that the compiler cannot count, and nothing waits in between: what waits for the
    // records would wait for the tile as well.  A push of 20 layers, batch 8, one worker 360 -> 349 us, 50 layers, batch 128 1565 -> 1546.
    const bool sub = PRE == 2 && C > 16 && half;                           // every second pixel of the shortcut
    const split::Buffer image = split::buffer(src + image_at, 4u * HW * HW * C);
    const split::Buffer image_beside = split::buffer(beside + (sub ? 2 : 1) * image_at, (sub ? 8u : 4u) * HW * HW * C);
#pragma unroll
    for (int e = 0; e < NL; ++e) {
        const unsigned at = (r_base + K::ROW0 - 1) * HW * C + e * STEP;
        val[e] = split::load4(image, inside(e) ? 4u * (at + 4 * tid) : split::OUTSIDE);
        if constexpr (PRE >= 2) {
            const bool in = inside(e) && !(sub && c4 >= C / 2);
            scv[e] = split::load4(image_beside, !in ? split::OUTSIDE : sub ? 4u * (2 * at + (2 * pr0 * HW + tid / V % HW) * C + c4) : 4u * (at + 4 * tid));
        }
    }
    // what the epilogue adds, masks with and sums over, a lane's four channels of its pixel of every tile: all these loads together (dst may
    // alias add, so the compiler cannot move them across the stores itself)
    float4 mu_c = make_float4(0.f, 0.f, 0.f, 0.f), is_c = mu_c, ga_c = mu_c, be_c = mu_c, addv[K::WM], maskv[POST ? K::WM : 1], xcv[POST ? K::WM : 1];
    constexpr int OUT_STEP = K::TROWS * HW * C;                                             // from tile to tile
    auto out_at_of = [&](const Role& r) -> unsigned {                                       // from the band's first pixel, first tile
        return ((r.row0 + K::TROWS * r.ks * K::WM) * HW + r.col) * C + r.co_w + 4 * r.q;
    };
    auto epilogue_loads = [&](const Role& r, int which = 7) {
        const unsigned at = out_at_of(r);
        if (POST && (which & 1)) {
            mu_c = *reinterpret_cast<const float4*>(post.stats + r.co_w + 4 * r.q);
            is_c = *reinterpret_cast<const float4*>(post.stats + C + r.co_w + 4 * r.q);
            if constexpr (REPEAT) {
                ga_c = *reinterpret_cast<const float4*>(post.gamma + r.co_w + 4 * r.q);
                be_c = *reinterpret_cast<const float4*>(post.beta + r.co_w + 4 * r.q);
            }
        }
#pragma unroll
        for (int wm = 0; wm < K::WM; ++wm) {
            if (!(which & 2)) ;
            else if constexpr (PL && POST)       // (a load behind a branch makes those before it wait: the compiler cannot count it)
                addv[wm] = split::load4(split::buffer(add + band_at, add ? 4u * R * HW * C : 0u), 4u * (at + wm * OUT_STEP));
            else
                addv[wm] = add ? load4(add + band_at + wm * OUT_STEP, at) : make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (POST) {
                if (!REPEAT && (which & 4)) maskv[wm] = load4(post.mask_src + band_at + wm * OUT_STEP, at);
                if (which & 1) xcv[wm] = load4(post.xc + band_at + wm * OUT_STEP, at);
            }
        }
    };
    // x halo tile of the fused d-filter: on its way during the epilogue
    float4 xin[WG && C != 64 ? NL : 1];
    const float* x_src = REPEAT ? post.xc : wg.x_in;
    auto load_x_tile = [&]() {
        if constexpr (C == 64) {            // this part's 16 channels
            xin[0] = load4(x_src + image_at, tid / 4 * C + part * K::CN + tid % 4 * 4);
            return;
        }
#pragma unroll
        for (int e = 0; e < NL; ++e) {
            if constexpr (SPREAD) {
                xin[e] = split::load4(split::buffer(x_src + image_at, 4u * HW * HW * C),
                                      inside(e) ? 4u * (unsigned)((r_base + K::ROW0 - 1) * HW * C + 4 * tid + e * STEP) : split::OUTSIDE);
                continue;
            }
            xin[e] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (inside(e)) xin[e] = load4(x_src + tile_at + e * STEP, 4u * tid);
        }
    };
    // REPEAT: the batch norm's four vectors for the x tile, in LDS (mean, invstd, gamma, beta)
    float* Sx = Sh + K::PS;
    // (stored behind the tile: here the store would wait for all loads before it, 349 -> 347.5 us)
    float x_norm = 0.f;
    if constexpr (WG && REPEAT) {
        static_assert(4 * C <= THREADS, "an element to a thread");
        if (tid < 4 * C) x_norm = (tid < 2 * C ? post.stats + tid : tid < 3 * C ? post.gamma + tid - 2 * C : post.beta + tid - 3 * C)[0];
    }
    auto x_value = [&](float4 o, int c) {       // of the x tile, inside the image
        if constexpr (REPEAT) {
            const float4 mu = *reinterpret_cast<const float4*>(Sx + c), is = *reinterpret_cast<const float4*>(Sx + C + c);
            const float4 ga = *reinterpret_cast<const float4*>(Sx + 2 * C + c), be = *reinterpret_cast<const float4*>(Sx + 3 * C + c);
            o.x = fmaxf(fmaf((o.x - mu.x) * is.x, ga.x, be.x), 0.f); o.y = fmaxf(fmaf((o.y - mu.y) * is.y, ga.y, be.y), 0.f);
            o.z = fmaxf(fmaf((o.z - mu.z) * is.z, ga.z, be.z), 0.f); o.w = fmaxf(fmaf((o.w - mu.w) * is.w, ga.w, be.w), 0.f);
        }
        return o;
    };
    if constexpr (K::EARLY && !SPREAD) {
        epilogue_loads(role_of(tid));
        if constexpr (WG) load_x_tile();
    }
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) split_filter(ky, 0);
    float* red = reinterpret_cast<float*>(lds);         // the tile is not there yet
    if constexpr (PRE == 1 || PRE == 2) {               // mean / invstd of the input
        if (parts) {
            const float nn = (float)pre.rows;
            Share* shares = reinterpret_cast<Share*>(red);
            static_assert(WAVES * C * sizeof(Share) <= K::XB, "room for the shares");
            const Share share = merge_lanes<C, THREADS>(rec, parts, nn, tid);
            if ((tid & 63) < C) shares[tid / 64 * C + tid % C] = share;
            __syncthreads();
            if (tid < C) {
                const float2 all = merge_waves<C, WAVES, K::RECORDS>(shares, parts, nn, tid);
                const float invstd = 1.0f / sqrtf(all.y / (float)pre.M + pre.eps);
                Sh[tid] = all.x;
                Sh[C + tid] = invstd;
                if (blockIdx.x == 0) { pre.stats_out[tid] = all.x; pre.stats_out[C + tid] = invstd; }
            }
        } else if (tid < 2 * C) {
            Sh[tid] = pre.stats_out[tid];
        }
        __syncthreads();
    }
    if constexpr (PRE == 3) {               // mean, invstd, gamma * invstd, sum(dz) / M, sum(dz * xhat) / M
        float sum_b = 0.f, sum_g = 0.f;
        if (parts) {
            float2* shares = reinterpret_cast<float2*>(red);
#pragma unroll
            for (int u = 1; u < K::RECORDS; ++u) { rec[0].x += rec[u].x; rec[0].y += rec[u].y; }
            sum_b = lanes_sum<C>(rec[0].x);
            sum_g = lanes_sum<C>(rec[0].y);
            if ((tid & 63) < C) shares[tid / 64 * C + tid % C] = make_float2(sum_b, sum_g);
            __syncthreads();
            if (tid < C) {
                sum_b = sum_g = 0.f;
#pragma unroll
                for (int w = 0; w < WAVES; ++w) { sum_b += shares[w * C + tid].x; sum_g += shares[w * C + tid].y; }
            }
        } else if (tid < C) {
            sum_b = bwd.totals[tid];
            sum_g = bwd.totals[C + tid];
        }
        if (tid < C) {
            const float is = norm_is;
            Sh[tid] = norm_mean;
            Sh[C + tid] = is;
            Sh[2 * C + tid] = norm_gamma * is;
            Sh[3 * C + tid] = sum_b * bwd.inv_m;
            Sh[4 * C + tid] = sum_g * bwd.inv_m;
            if (parts && blockIdx.x == 0) { bwd.dbeta[tid] = sum_b; bwd.dgamma[tid] = sum_g; }
        }
        __syncthreads();
    }
    if constexpr (PL) first_columns();          // behind the records of every wavefront: they are needed first (50 layers, batch 128 1698 -> 1688 us)
    auto stage = [&](char* to, float4 v) {  // 4 channels of a pixel as their three terms
        uint2 pl[split::PLANES];
        split::split4(split::scaled(v), pl);
#pragma unroll
        for (int p = 0; p < split::PLANES; ++p) *reinterpret_cast<uint2*>(to + p * K::PLANE) = pl[p];
    };
    // what the convolution runs on, four channels of a pixel of src (and of the shortcut or xc); the batch norm's vectors of these channels
    struct Vectors { float4 mu, is, ga, be, dg; };
    auto vectors = [&](int c, bool own_channels) {
        Vectors v{};
        if constexpr (PRE == 3) {
            v.ga = *reinterpret_cast<const float4*>(Sh + 2 * C + c);            // gamma * invstd
            v.be = *reinterpret_cast<const float4*>(Sh + 3 * C + c);
            v.dg = *reinterpret_cast<const float4*>(Sh + 4 * C + c);
        }
        if constexpr (PRE == 1 || PRE == 2) {
            v.ga = own_channels ? norm_g : *reinterpret_cast<const float4*>(norm_first + c);
            v.be = own_channels ? norm_b : *reinterpret_cast<const float4*>(norm_second + c);
        }
        if constexpr (PRE != 0) {
            v.mu = *reinterpret_cast<const float4*>(Sh + c);
            v.is = *reinterpret_cast<const float4*>(Sh + C + c);
        }
        return v;
    };
    auto transformed = [&](float4 o, float4 sc, const Vectors& v) {
        if constexpr (PRE == 3) {
            o.x = v.ga.x * (o.x - v.be.x - (sc.x - v.mu.x) * v.is.x * v.dg.x);
            o.y = v.ga.y * (o.y - v.be.y - (sc.y - v.mu.y) * v.is.y * v.dg.y);
            o.z = v.ga.z * (o.z - v.be.z - (sc.z - v.mu.z) * v.is.z * v.dg.z);
            o.w = v.ga.w * (o.w - v.be.w - (sc.w - v.mu.w) * v.is.w * v.dg.w);
        }
        if constexpr (PRE == 1 || PRE == 2) {
            o.x = fmaf((o.x - v.mu.x) * v.is.x, v.ga.x, v.be.x);
            o.y = fmaf((o.y - v.mu.y) * v.is.y, v.ga.y, v.be.y);
            o.z = fmaf((o.z - v.mu.z) * v.is.z, v.ga.z, v.be.z);
            o.w = fmaf((o.w - v.mu.w) * v.is.w, v.ga.w, v.be.w);
            if constexpr (PRE == 2) { o.x += sc.x; o.y += sc.y; o.z += sc.z; o.w += sc.w; }
            o.x = fmaxf(o.x, 0.f); o.y = fmaxf(o.y, 0.f); o.z = fmaxf(o.z, 0.f); o.w = fmaxf(o.w, 0.f);
        }
        return o;
    };
    auto input = [&](int h, int w, int c) {  // the same from memory, zero outside the image
        if (h < 0 || h >= HW || w < 0 || w >= HW) return make_float4(0.f, 0.f, 0.f, 0.f);
        const long off = image_at + (h * HW + w) * C + c;
        float4 sc = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (PRE == 2) {
            if (!(C > 16 && half)) sc = *reinterpret_cast<const float4*>(beside + off);
            else if (c < C / 2) sc = *reinterpret_cast<const float4*>(beside + 2 * image_at + (2 * h * HW + w) * C + c);
        }
        if constexpr (PRE == 3) sc = *reinterpret_cast<const float4*>(beside + off);
        return transformed(*reinterpret_cast<const float4*>(src + off), sc, vectors(c, false));
    };
    if constexpr (WG && C == 64)            // the x tile's border
        for (int i = tid; i < 4 * (K::TW - 1) * (K::X2PITCH / 8); i += THREADS) {
            const int px = i / (K::X2PITCH / 8), side = px / (K::TW - 1), j = px % (K::TW - 1);
            const int r = side == 0 ? 0 : side == 1 ? K::TW - 1 : side == 2 ? j + 1 : j, c = side == 0 ? j : side == 1 ? j + 1 : side == 2 ? 0 : K::TW - 1;
            *reinterpret_cast<uint2*>(lds + K::LDS_X + (r * K::TW + c) * K::X2PITCH + 8 * (i % (K::X2PITCH / 8))) = make_uint2(0u, 0u);
        }
    for (int i = tid; i < K::ZERO; i += THREADS) {          // outside the image: left and right, for a whole image above and below
        const int px = i / K::ZERO_UNITS, unit = i % K::ZERO_UNITS;
        int r = px >> 1, c = (px & 1) * (K::TW - 1);
        if (K::WHOLE && px >= 2 * (R + 2)) { r = (px & 1) * (R + 1); c = ((px - 2 * (R + 2)) >> 1) + 1; }
        char* to = Xs + r * K::ROW + c * K::PITCH + unit * K::ZERO_UNIT;
        if constexpr (K::ZERO_UNIT == 16) *reinterpret_cast<uint4*>(to) = make_uint4(0u, 0u, 0u, 0u);
        else *reinterpret_cast<uint2*>(to) = make_uint2(0u, 0u);
    }
    const Vectors own_vectors = vectors(c4, true);
#pragma unroll
    for (int e = 0; e < NL; ++e) {
        if (!own(e)) continue;
        if constexpr (PRE != 0) {
            if (inside(e)) {
                val[e] = transformed(val[e], scv[PRE >= 2 ? e : 0], own_vectors);
                // the band's own rows (not the halo rows) are this workgroup's part of `a` or dx
                if (!WG && part == 0 && (K::WHOLE || (pr0 + e * RE >= 1 && pr0 + e * RE <= R)))
                    *reinterpret_cast<float4*>((PRE == 3 ? bwd.dx_out : pre.act_out) + tile_at + e * STEP + 4u * tid) = val[e];
            }
        }
        stage(tile_to + e * STEP_TO, val[e]);
    }
    if constexpr (WG && REPEAT)
        if (tid < 4 * C) Sx[tid] = x_norm;
    __syncthreads();

    // ---- products.  Pixel operand (st, kx): the tile that starts st rows below the wavefront's first one, kx to the right
    //      (halo coordinates); it meets filter row ky in the tile t with TROWS t + ky = st.
    floatx4 acc[K::WM];
    {
        constexpr int NT = K::NT, LAST = (NT - 1) * K::TROWS, ST = LAST + 3;
        const Role r = role_of(tid);
        int at_px = r.row0 * K::ROW + r.col * K::PITCH + (C == 16 ? 8 : 16) * r.q + 64 * r.ks;
        const char* base = Xs + at_px;
        if constexpr (C == 16) asm("" : "+v"(at_px));
        const char* again = Xs + at_px;
        // Two accumulators: the leading products, and the small ones (2^-8 and less of them), so that most of the roundings are
        // those of the small sum.
        floatx4 a[NT], lo[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) a[t] = lo[t] = floatx4{0.f, 0.f, 0.f, 0.f};
        split::Pix<C> x[2];
        auto pixels = [&](int i) { return split::pixel_operand<C, K::PLANE>(base + i % ST * K::ROW + i / ST * K::PITCH, again + i % ST * K::ROW + i / ST * K::PITCH); };
        x[0] = pixels(0);
#pragma unroll
        for (int i = 0; i < 3 * ST; ++i) {
            const int st = i % ST, kx = i / ST;
            // filter row ky meets its last pixel operand of a column at st = LAST + ky: there the next column's is fetched one
            // step before and split one step after
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                if (i % ST == (LAST + ky + 1) % ST && kx + (ky < 2) >= 1 && kx + (ky < 2) <= 2) split_filter(ky, kx + (ky < 2));
                if (!PL && COLUMNS == 1 && st == LAST + ky - 1 && kx < 2) load_filter(ky, kx + 1);
            }
            if constexpr (PL && C == 16)                // the quad that is not stored, for the row that this step is the first to use
                if (st < 3) {
                    split::Filt<C>& f = filt[kx % COLUMNS][st];
                    f.v[1] = make_uint4(f.v[2].z, f.v[2].w, f.v[2].x, f.v[2].y);
                }
            if (i + 1 < 3 * ST) x[(i + 1) & 1] = pixels(i + 1);
            __builtin_amdgcn_sched_barrier(0);      // or the compiler moves the reads down to their use, behind the products
#pragma unroll
            for (int p = 0; p < split::products<C>(); ++p)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int ky = st - K::TROWS * t;
                    if (ky < 0 || ky > 2) continue;
                    floatx4& to = p + 1 < split::products<C>() ? lo[t] : a[t];
                    to = split::product<C>(p, filt[PL ? kx % COLUMNS : 0][ky], x[i & 1], to);
                }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (SPREAD) {
                if (st < 3 && kx < 2) load_filter(st, kx + 1);
                if (st == 3 && kx == 0) epilogue_loads(r);
                if constexpr (WG)
                    if (st == 3 && kx == 1) load_x_tile();
            }
            if constexpr (PL && COLUMNS == 1)        // into the registers of the row that has just been used for the last time
            {
                if (st >= LAST && kx < 2) load_filter(st - LAST, kx + 1);
                // What the epilogue reads, as far as the registers that the last column's rows leave go (all of it with 16 and 32 channels: up
                // to 35 spilled).  Epilogue of the last stage 2400 to 3700 -> 750 cycles; a push of 50 layers, batch 128, one worker 1661 -> 1650 us.
                if constexpr (C == 64) {
                    if (st >= LAST && kx == 2) epilogue_loads(r, 1 << (st - LAST));
                } else {
                    if (st == LAST + (REPEAT ? 1 : 2) && kx == 2) epilogue_loads(r, 1);
                }
            }
        }
        mma::drain();
#pragma unroll
        for (int t = 0; t < NT; ++t) a[t] += lo[t];
        if constexpr (K::KS == 1) {
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = a[t];
        } else {
            // the two wavefronts of a group of pixels hold partial sums over their halves of the input channels: each
            // hands the other the two tiles it will not finish and adds what it receives (first half + second half)
            const int ks = r.ks, lane = r.lane, wave = r.wave;
            if constexpr (!WG) __syncthreads();            // every wavefront has read the tile for the last time
            float* Ex = reinterpret_cast<float*>(WG ? lds + K::LDS_X + K::X2 : lds);       // [wavefront][WM][64][4]
#pragma unroll
            for (int wm = 0; wm < K::WM; ++wm)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float give = ks == 0 ? a[K::WM + wm][v] : a[wm][v];
                    acc[wm][v] = ks == 0 ? a[wm][v] : a[K::WM + wm][v];
                    Ex[((wave * K::WM + wm) * 64 + lane) * 4 + v] = give;
                }
            __syncthreads();
            const int partner = (r.wave_m ^ 1) * K::WAVES_N + r.wave_n;
#pragma unroll
            for (int wm = 0; wm < K::WM; ++wm)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[wm][v] += Ex[((partner * K::WM + wm) * 64 + lane) * 4 + v];
        }
    }

    if constexpr (WARM) asm volatile("" :: "v"(warm));
    int again_tid = tid;
    asm("" : "+v"(again_tid));
    const Role role = role_of(again_tid);
    const int l16 = role.l16, q = role.q, wave = role.wave, lane = role.lane, wave_n = role.wave_n, wave_m = role.wave_m, co_w = role.co_w;
    const int ks = role.ks, row0 = role.row0, col = role.col;
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
    const unsigned out_at = out_at_of(role);
    if constexpr (!K::EARLY) {
        epilogue_loads(role, !PL ? 7 : C == 64 ? 0 : 6);
        if constexpr (WG) load_x_tile();
    }
    float4 sum_dz = make_float4(0.f, 0.f, 0.f, 0.f), sum_dzx = sum_dz;
#pragma unroll
    for (int wm = 0; wm < K::WM; ++wm) {
        float4 r = make_float4(acc[wm][0] + addv[wm].x, acc[wm][1] + addv[wm].y, acc[wm][2] + addv[wm].z, acc[wm][3] + addv[wm].w);
        if constexpr (POST) {
            const float4 hat = make_float4((xcv[wm].x - mu_c.x) * is_c.x, (xcv[wm].y - mu_c.y) * is_c.y, (xcv[wm].z - mu_c.z) * is_c.z, (xcv[wm].w - mu_c.w) * is_c.w);
            if constexpr (REPEAT)
                maskv[wm] = make_float4(fmaf(hat.x, ga_c.x, be_c.x), fmaf(hat.y, ga_c.y, be_c.y), fmaf(hat.z, ga_c.z, be_c.z), fmaf(hat.w, ga_c.w, be_c.w));
            r.x = maskv[wm].x > 0.f ? r.x : 0.f; r.y = maskv[wm].y > 0.f ? r.y : 0.f;
            r.z = maskv[wm].z > 0.f ? r.z : 0.f; r.w = maskv[wm].w > 0.f ? r.w : 0.f;
            sum_dz.x += r.x; sum_dz.y += r.y; sum_dz.z += r.z; sum_dz.w += r.w;
            sum_dzx.x = fmaf(r.x, hat.x, sum_dzx.x); sum_dzx.y = fmaf(r.y, hat.y, sum_dzx.y);
            sum_dzx.z = fmaf(r.z, hat.z, sum_dzx.z); sum_dzx.w = fmaf(r.w, hat.w, sum_dzx.w);
        }
        *reinterpret_cast<float4*>(dst + band_at + wm * OUT_STEP + out_at) = r;
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
        put(Ss + K::SC, sum16(sum_dzx));
        __syncthreads();
        if (wave_m == 0 && l16 == 0) put_records(post.records, tile_total(Ss), tile_total(Ss + K::SC));
    }
    // ---- fused d-filter of the same layer:
    //      dw[tap][ci][co] += x[pixel + tap][ci] dx[pixel][co], pixels as reduction index, 32 to an MFMA, both operands
    //      by transposing reads.  The dx operands go to registers, the x tile takes the place of the dx tile: half the LDS, so that
    //      another workgroup fits beside this one.  A run of 32 pixels is one image row (C = 16) or two (C = 32); an x operand
    //      fetched for one filter row serves the run above it too.  Rows of the matrix-core tile: co, columns: ci.
    //      One filter column after the other, its small products with accumulators of their own: in one
    //      accumulator all six are rounded to the size of the sum, and with a bias, so that the error of the sum over the workgroups
    //      grew with their number (16 channels, batch 1 / 37 / 128: 1.1e-7 / 2.0e-7 / 3.2e-7; so 0.7e-7 / 1.0e-7 / 1.2e-7).
    if constexpr (WG && C != 64) {
        constexpr int RUNS = K::RUNS, RROWS = 32 / HW;         // image rows per run
        const int cit = C == 16 ? 0 : (wave & 3) >> 1, cot = C == 16 ? 0 : wave & 1;
        const int first = RUNS * RROWS * (wave / K::DTILES);   // first image row of the wavefront's runs
        const char* xa[2];                                     // of pixels 8 q + 4 h + l16 / 4 of the first run
        uint4 d[RUNS][split::PLANES];
        {
            const char* da[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int p = 8 * q + 4 * h + (l16 >> 2);
                const int o = (first + p / HW) * K::ROW + p % HW * K::PITCH + 8 * (l16 & 3);
                xa[h] = Xs + o + 32 * cit;
                da[h] = Xs + o + K::ROW + K::PITCH + 32 * cot;
            }
#pragma unroll
            for (int run = 0; run < RUNS; ++run)
                split::transposed_operand<K::PLANE>(d[run], da[0] + run * RROWS * K::ROW, da[1] + run * RROWS * K::ROW);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < NL; ++e)
            if (own(e)) stage(tile_to + e * STEP_TO, !REPEAT ? xin[e] : inside(e) ? x_value(xin[e], c4) : make_float4(0.f, 0.f, 0.f, 0.f));
        __syncthreads();
        constexpr int ST = RROWS * (RUNS - 1) + 3;             // image rows the runs and the three filter rows meet
        constexpr int XB = WAVES == 8 ? 1 : 2;                  // operands in registers: four wavefronts a SIMD hide the fetch
        uint4 x[XB][split::PLANES];
        auto load_x = [&](int b, int i) {
            const int off = i % ST * K::ROW + i / ST * K::PITCH;
            split::transposed_operand<K::PLANE>(x[b], xa[0] + off, xa[1] + off);
        };
        floatx4 dw[C == 16 ? 9 : 1];                           // C = 16: all taps, summed over the wavefronts at the end
        floatx4* Column = reinterpret_cast<floatx4*>(lds + K::LDS_X) + (wave & 3) * 3 * 64 + lane;
        float* pout = wg.partial + (long)tile * 9 * C * C;
        float worst = 0.f;
        // C = 32: the sums of a filter column go to memory, with eight wavefronts those of both halves of the image: 4 to 7 hand theirs to 0 to 3
        auto finish_column = [&](floatx4 (&v)[3], int kx) {
            if constexpr (K::RSPLIT == 2) {
                if (kx > 0) __syncthreads();                   // the column before has been read
                if (wave >= 4)
#pragma unroll
                    for (int ky = 0; ky < 3; ++ky) Column[64 * ky] = v[ky];
                __syncthreads();
                if (wave < 4)
#pragma unroll
                    for (int ky = 0; ky < 3; ++ky) v[ky] += Column[64 * ky];
            }
            if (K::RSPLIT == 1 || wave < 4)
#pragma unroll
                for (int ky = 0; ky < 3; ++ky)
                    *reinterpret_cast<floatx4*>(pout + ((3 * ky + kx) * C + 16 * cit + l16) * C + 16 * cot + 4 * q) = v[ky];
        };
        if constexpr (XB == 2) load_x(0, 0);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            floatx4 lead[3], small[3];
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) lead[ky] = small[ky] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < ST; ++st) {
                const int i = ST * kx + st;
                if constexpr (XB == 1) load_x(0, i);
                else if (i + 1 < 3 * ST) load_x((i + 1) & 1, i + 1);
                __builtin_amdgcn_sched_barrier(0);
                constexpr int PD[6] = {0, 2, 1, 0, 1, 0}, PX[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
                for (int p = 0; p < 6; ++p)
#pragma unroll
                    for (int run = 0; run < RUNS; ++run) {
                        const int ky = st - RROWS * run;
                        if (ky < 0 || ky > 2) continue;
                        floatx4& to = p < 5 ? small[ky] : lead[ky];
                        to = split::mfma(d[run][PD[p]], x[i % XB][PX[p]], to);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
            mma::drain();
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                lead[ky] += small[ky];
                worst = split::spoil(lead[ky], worst);
                lead[ky] *= split::UNSCALE;
            }
            if constexpr (C == 16) {
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) dw[3 * ky + kx] = lead[ky];
            } else {
                finish_column(lead, kx);
            }
        }
        // sums beyond the range of the scaled terms: the wavefront's runs from the operands in memory, four pixels of a row a step (C = 32:
        // all of the workgroup's, which meet in finish_column)
        bool again = split::spoiled(worst);
        if constexpr (C != 16) {                               // (through the column sums' place: __syncthreads_or takes LDS of its own, too much for two
            if (lane == 0) Ss[wave] = again ? 1.f : 0.f;       // workgroups of 16x16 pixels and 32 channels to a compute unit)
            __syncthreads();
#pragma unroll
            for (int j = 0; j < WAVES; ++j) again |= Ss[j] != 0.f;
        }
        if (again) {
#pragma unroll 1
            for (int kx = 0; kx < 3; ++kx) {
                floatx4 v[3];
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) v[ky] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int p = first * HW + q; p < (first + RUNS * RROWS) * HW; p += 4) {
                    const int h = r_base + p / HW, w = p % HW, c = 16 * cot + l16;
                    const float4 dx = input(h, w, c & ~3);
                    const float dv[1] = {c & 2 ? (c & 1 ? dx.w : dx.z) : (c & 1 ? dx.y : dx.x)};
#pragma unroll
                    for (int ky = 0; ky < 3; ++ky) {
                        const int xh = h + ky - 1, xw = w + kx - 1;
                        const bool in = (unsigned)xh < (unsigned)HW && (unsigned)xw < (unsigned)HW;
                        const float xv[1] = {in ? wg.x_in[(((long)n * HW + xh) * HW + xw) * C + 16 * cit + l16] : 0.f};
                        v[ky] = split::product32(dv, xv, v[ky]);
                    }
                }
                mma::drain();
                if constexpr (C == 16) {
#pragma unroll
                    for (int t = 0; t < 9; ++t)
                        if (t % 3 == kx) dw[t] = v[t / 3];
                } else {
                    finish_column(v, kx);
                }
            }
        }
        if constexpr (C == 16) {
            __syncthreads();                                  // the tile is no longer needed: the wavefronts' partial sums in its place
            floatx4* Red = reinterpret_cast<floatx4*>(lds);       // [wavefront][tap][ci][co / 4]
            constexpr int E4 = 9 * C * C / 4;
#pragma unroll
            for (int t = 0; t < 9; ++t) Red[wave * E4 + (t * C + l16) * 4 + q] = dw[t];
            __syncthreads();
            for (int idx = tid; idx < E4; idx += THREADS) {
                floatx4 s_[WAVES / 4];
#pragma unroll
                for (int j = 0; j < WAVES / 4; ++j)
                    s_[j] = (Red[4 * j * E4 + idx] + Red[(4 * j + 1) * E4 + idx]) + (Red[(4 * j + 2) * E4 + idx] + Red[(4 * j + 3) * E4 + idx]);
                if constexpr (WAVES == 8) s_[0] += s_[1];
                reinterpret_cast<floatx4*>(pout)[idx] = s_[0];
            }
        }
    }

    // The same with 64 channels: a wavefront owns 16 output channels, all nine taps of this part's 16 input channels and the image's two runs of
    // 32 pixels (four rows each); the dx tile stays where it is.  Products and
    // sums in the order of wgrad3x3_wide_kernel, which as a launch of its own takes 8.5 us at these batches, this 2.  With that kernel / so, a round
    // of pushes, us: 20 layers, batch 8, four workers 652 / 606, batch 17, three 577 / 537; 50 layers, batch 8, two 1059 / 979; 110 layers, batch 3,
    // eight 7177 / 6054.  (Partial sums of an image are nine times its activations: not for larger batches.)
    if constexpr (WG && C == 64) {
        constexpr int RUN = 4 * K::TW;                         // pixels of the tile from run to run
        char* X2 = lds + K::LDS_X;
        {
            const int px = tid / 4;
            uint2 pl[split::PLANES];
            split::split4(split::scaled(x_value(xin[0], part * K::CN + tid % 4 * 4)), pl);
#pragma unroll
            for (int p = 0; p < split::PLANES; ++p)
                *reinterpret_cast<uint2*>(X2 + ((px / HW + 1) * K::TW + px % HW + 1) * K::X2PITCH + p * K::X2PLANE + 8 * (tid % 4)) = pl[p];
        }
        const char *xa[2], *da[2];                             // of pixels 8 q + 4 h + l16 / 4 of the first run
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int p = 8 * q + 4 * h + (l16 >> 2);
            xa[h] = X2 + (p / HW * K::TW + p % HW) * K::X2PITCH + 8 * (l16 & 3);
            da[h] = Xs + (p / HW + 1) * K::ROW + (p % HW + 1) * K::PITCH + 32 * wave + 8 * (l16 & 3);
        }
        uint4 d[2][split::PLANES], x[2][split::PLANES];
#pragma unroll
        for (int run = 0; run < 2; ++run) split::transposed_operand<K::PLANE>(d[run], da[0] + run * 4 * K::ROW, da[1] + run * 4 * K::ROW);
        auto load_x = [&](int i) {                             // filter column i / 6, run i / 3 mod 2, row i mod 3
            const int off = (i / 3 % 2 * RUN + i % 3 * K::TW + i / 6) * K::X2PITCH;
            split::transposed_operand<K::X2PLANE>(x[i & 1], xa[0] + off, xa[1] + off);
        };
        __syncthreads();
        load_x(0);
        const int ci = part * K::CN + l16;
        float* pout = wg.partial + (long)n * 9 * C * C + ci * C + 16 * wave + 4 * q;
        float worst = 0.f;
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            floatx4 sum[3];
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) sum[ky] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 6 * kx; i < 6 * kx + 6; ++i) {
                if (i + 1 < 18) load_x(i + 1);
                __builtin_amdgcn_sched_barrier(0);
                constexpr int PD[6] = {0, 2, 1, 0, 1, 0}, PX[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
                for (int p = 0; p < 6; ++p) sum[i % 3] = split::mfma(d[i / 3 % 2][PD[p]], x[i & 1][PX[p]], sum[i % 3]);
                __builtin_amdgcn_sched_barrier(0);
            }
            mma::drain();
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                worst = split::spoil(sum[ky], worst);
                *reinterpret_cast<floatx4*>(pout + (3 * ky + kx) * C * C) = sum[ky] * split::UNSCALE;
            }
        }
        if (split::spoiled(worst)) {    // beyond the range of the scaled terms: from the operands in memory, four pixels of a row a step
            const int c = 16 * wave + l16;
#pragma unroll 1
            for (int tap = 0; tap < 9; ++tap) {
                floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int p = q; p < HW * HW; p += 4) {
                    const int h = p / HW, w = p % HW, xh = h + tap / 3 - 1, xw = w + tap % 3 - 1;
                    const float4 dx = input(h, w, c & ~3);
                    const float dv[1] = {c & 2 ? (c & 1 ? dx.w : dx.z) : (c & 1 ? dx.y : dx.x)};
                    const bool in = (unsigned)xh < (unsigned)HW && (unsigned)xw < (unsigned)HW;
                    const float xv[1] = {in ? wg.x_in[image_at + (xh * HW + xw) * C + ci] : 0.f};
                    v = split::product32(dv, xv, v);
                }
                mma::drain();
                *reinterpret_cast<floatx4*>(pout + tap * C * C) = v;
            }
        }
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
        put(Ss + K::SC, sum16(s_));
        __syncthreads();
        if (wave_m == 0 && l16 == 0) put_records(bn_partial, mean, tile_total(Ss + K::SC));
    }
}

template <bool PL, int C, int HW, int R, int NSPLIT, int WAVES, bool T, int PRE, bool POST, bool WG, bool REPEAT = false>
int launch_form(hipStream_t s, const float* src, const Filter3x3& w, const float* add, float* dst, float* bn_partial, int N,
           const PreBn& pre, const PostBn& post, const BwdBn& bwd, const jobs::ReduceJob& rj, const WgradFused& wg) {
    using K = Cfg<C, HW, R, NSPLIT, WAVES>;
    constexpr size_t LDS_BYTES = WG ? K::LDS_BYTES_WG : K::LDS_BYTES;
    static_assert(LDS_BYTES >= jobs::LDS_FLOATS * (K::THREADS / jobs::THREADS) * sizeof(float), "room for a carried job");
    static bool attr_set = false;       // raise the dynamic-LDS limit once per instantiation
    auto kern = conv3x3_kernel<C, HW, R, NSPLIT, WAVES, T, PRE, POST, WG, PL, REPEAT>;
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)LDS_BYTES) != hipSuccess)
            return -1;
        attr_set = true;
    }
    const int conv_blocks = N * (HW / R) * NSPLIT;
    const int list = PRE == 3 ? bwd.totals ? 0 : bwd.parts : (pre.merge ? pre.parts : 0) | (pre.half ? 1 << 16 : 0);
    const PreArgs& pre_args = pre;
    const BwdArgs& bwd_args = bwd;
    hipLaunchKernelGGL(kern, dim3(conv_blocks + rj.blocks), dim3(K::THREADS), LDS_BYTES, s, PRE == 3 ? bwd.records : pre.records, list, conv_blocks, src,
                       PRE == 3 ? bwd.xc : pre.shortcut, w.planes, PRE == 3 ? bwd.stats : pre.gamma, PRE == 3 ? bwd.gamma : pre.beta, w.w, add, dst,
                       bn_partial, pre_args, post, bwd_args, rj, wg);
    return (int)hipGetLastError();
}

template <int C, int HW, int R, int NSPLIT, int WAVES, bool T, int PRE = 0, bool POST = false, bool WG = false>
int launch(hipStream_t s, const float* src, const Filter3x3& w, const float* add, float* dst, float* bn_partial, int N, const PreBn& pre = PreBn{},
           const PostBn& post = PostBn(), const BwdBn& bwd = BwdBn(), const jobs::ReduceJob& rj = jobs::ReduceJob(), const WgradFused& wg = WgradFused()) {
    // what a network's step launches (with 16 and 32 channels d-input and d-filter always come from one kernel)
    if constexpr (T && PRE == 3 && (WG || C == 64))
        if (w.planes && post.gamma)
            return launch_form<true, C, HW, R, NSPLIT, WAVES, T, PRE, POST, WG, true>(s, src, w, add, dst, bn_partial, N, pre, post, bwd, rj, wg);
    if constexpr (!T || (PRE == 3 && (WG || C == 64)))
        if (w.planes) return launch_form<true, C, HW, R, NSPLIT, WAVES, T, PRE, POST, WG>(s, src, w, add, dst, bn_partial, N, pre, post, bwd, rj, wg);
    return launch_form<false, C, HW, R, NSPLIT, WAVES, T, PRE, POST, WG>(s, src, w, add, dst, bn_partial, N, pre, post, bwd, rj, wg);
}

// The reduction job a launch carries, and the workgroups (of `threads` threads) given to it.
inline jobs::ReduceJob reduce_job(const jobs::Partials& waiting, int threads) {
    jobs::ReduceJob rj = jobs::ReduceJob();
    if (waiting.partial) {
        static_cast<jobs::Partials&>(rj) = waiting;
        const int groups = jobs::reduce_groups(rj.E, rj.chunks), per = threads / jobs::THREADS;
        rj.blocks = ((groups < 288 ? groups : 288) + per - 1) / per;
    }
    return rj;
}

}  // namespace
