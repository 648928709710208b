// Fully connected layers: C = op(A) * op(B) (+ bias) (ReLU), fp32 on the matrix cores.
// Operands come in through generic strides, so the same product serves y = x W (+b), dx = dy W^T and
// dW = x^T dy of Alg. 1's worker gradient.
//
// These products are small (0.005 to 1 GFLOP) and bound by latency, not by the matrix cores or by memory: what counts is
// how many loads are in flight.  So there is no LDS staging and no barrier in the product: a wavefront fetches its MFMA
// operands straight from memory into registers, G k-chunks of 16 at a time, the next G already in flight while the matrix
// cores work on the present ones, and the wavefronts of a workgroup split the reduction index of one output tile (their
// partial tiles are summed through LDS once, in a fixed order).  Measured, kernel time: 32 x 256 with K = 3072 17 us (93 us
// when workgroups of 64x64 tiles walked the reduction one 16-wide LDS stage and barrier after the other, on four compute
// units); 128 x 384 with K = 3136 17 us in one kernel (22 us with 22 layers of K and a second kernel that sums them).
#include <mutex>

#include "mma.hpp"
#include "../../include/dssp_kernels.h"

namespace {

struct Operand {
    const float* p;     // element (i, k) at p[i * s + k * ks], i = row of op(A) / column of op(B)
    long s, ks;
};

// acc += (rows row0 .. of a) * (columns col0 .. of b) over the k-chunks first, first + every, ... of [0, K).
//   AV / BV: the operand is contiguous along k, 16-byte aligned with a stride and K that are multiples of 4 (one 16-byte
//   load per lane and chunk); otherwise four scalar loads, which coalesce across the lanes when i is the contiguous index.
// Rows and columns beyond M / N are clamped (the caller drops those results), k beyond K reads as zero.
template <int WM, int WN, int G, bool AV, bool BV>
__device__ __forceinline__ void wave_product(const Operand& a, const Operand& b, int M, int N, int row0, int col0, int K, int first,
                                             int every, floatx4 (&acc)[WM][WN], int lane) {
    const int l16 = lane & 15, q = lane >> 4;
    const float *pa[WM], *pb[WN];
#pragma unroll
    for (int w = 0; w < WM; ++w) pa[w] = a.p + (long)min(row0 + 16 * w + l16, M - 1) * a.s;
#pragma unroll
    for (int w = 0; w < WN; ++w) pb[w] = b.p + (long)min(col0 + 16 * w + l16, N - 1) * b.s;
    const int chunks = (K + mma::KC - 1) / mma::KC;
    float fa[2][G][WM][4], fb[2][G][WN][4];
    auto fetch = [&](int buf, int c0) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int c = c0 + u * every;
            if (c >= chunks) {                          // uniform over the wavefront
#pragma unroll
                for (int s = 0; s < 4; ++s) {
#pragma unroll
                    for (int w = 0; w < WM; ++w) fa[buf][u][w][s] = 0.f;
#pragma unroll
                    for (int w = 0; w < WN; ++w) fb[buf][u][w][s] = 0.f;
                }
                continue;
            }
            const int k = c * mma::KC + 4 * q;
            if (AV && BV ? true : c * mma::KC + mma::KC <= K) {
                // with K a multiple of 4 a lane's four k are all inside or all outside
                const bool in = !(AV && BV) || k < K;
                const int kc = in ? k : 0;
#pragma unroll
                for (int w = 0; w < WM; ++w) {
                    if constexpr (AV) {
                        const float4 v = *reinterpret_cast<const float4*>(pa[w] + kc);
                        fa[buf][u][w][0] = in ? v.x : 0.f; fa[buf][u][w][1] = in ? v.y : 0.f;
                        fa[buf][u][w][2] = in ? v.z : 0.f; fa[buf][u][w][3] = in ? v.w : 0.f;
                    } else {
#pragma unroll
                        for (int s = 0; s < 4; ++s) fa[buf][u][w][s] = pa[w][(long)(kc + s) * a.ks];
                    }
                }
#pragma unroll
                for (int w = 0; w < WN; ++w) {
                    if constexpr (BV) {
                        const float4 v = *reinterpret_cast<const float4*>(pb[w] + kc);
                        fb[buf][u][w][0] = in ? v.x : 0.f; fb[buf][u][w][1] = in ? v.y : 0.f;
                        fb[buf][u][w][2] = in ? v.z : 0.f; fb[buf][u][w][3] = in ? v.w : 0.f;
                    } else {
#pragma unroll
                        for (int s = 0; s < 4; ++s) fb[buf][u][w][s] = pb[w][(long)(kc + s) * b.ks];
                    }
                }
            } else {                                    // the partial last chunk
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const bool in = k + s < K;
                    const long kk = in ? k + s : 0;
#pragma unroll
                    for (int w = 0; w < WM; ++w) { const float v = pa[w][kk * a.ks]; fa[buf][u][w][s] = in ? v : 0.f; }
#pragma unroll
                    for (int w = 0; w < WN; ++w) { const float v = pb[w][kk * b.ks]; fb[buf][u][w][s] = in ? v : 0.f; }
                }
            }
        }
    };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[buf][u][i][s], fb[buf][u][j][s], acc[i][j], 0, 0, 0);
    };
    if (first >= chunks) return;
    fetch(0, first);
    for (int c = first; c < chunks; c += 2 * G * every) {
        if (c + G * every < chunks) fetch(1, c + G * every);
        multiply(0);
        if (c + G * every >= chunks) break;
        if (c + 2 * G * every < chunks) fetch(0, c + 2 * G * every);
        multiply(1);
    }
}

struct Epilogue {
    float* C;                   // element (i, j) at C[i * ldc + j]
    long ldc;
    const float* bias;          // [N] or null
    int relu;
    const float* mask;          // laid out as C, or null: the result is 0 where mask <= 0
};

__device__ __forceinline__ void store_result(const Epilogue& e, int row, int col, float x) {
    if (e.bias) x += e.bias[col];
    if (e.relu) x = fmaxf(x, 0.f);
    if (e.mask) x = e.mask[(long)row * e.ldc + col] > 0.f ? x : 0.f;
    e.C[(long)row * e.ldc + col] = x;
}

// One output tile by a workgroup of GM x GN x KW wavefronts, each 16 WM x 16 WN outputs of it; the KW wavefronts of an
// output sub-tile take its k-chunks in turn.  lds: KW * GM * GN * 256 * WM * WN floats if KW > 1.
template <int WM, int WN, int GM, int GN, int G, bool AV, bool BV>
__device__ __forceinline__ void tile_product(const Operand& a, const Operand& b, int M, int N, int K, int tile_m, int tile_n,
                                             const Epilogue& e, float* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kw = blockDim.x / (64 * GM * GN), sub = wave % (GM * GN), part = wave / (GM * GN);
    const int row0 = (tile_m * GM + sub / GN) * 16 * WM, col0 = (tile_n * GN + sub % GN) * 16 * WN;
    floatx4 acc[WM][WN];
    mma::zero(acc);
    wave_product<WM, WN, G, AV, BV>(a, b, M, N, row0, col0, K, part, kw, acc, lane);
    mma::drain();
    const int l16 = lane & 15, q = lane >> 4;
    if (kw == 1) {
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = row0 + 16 * i + 4 * q + v, col = col0 + 16 * j + l16;
                    if (row < M && col < N) store_result(e, row, col, acc[i][j][v]);
                }
        return;
    }
    constexpr int TILE = 256 * WM * WN, ALL = TILE * GM * GN;
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                lds[part * ALL + sub * TILE + (16 * i + 4 * q + v) * 16 * WN + 16 * j + l16] = acc[i][j][v];
    __syncthreads();
    for (int idx = threadIdx.x; idx < ALL; idx += blockDim.x) {
        float s = 0.f;
        for (int p = 0; p < kw; ++p) s += lds[p * ALL + idx];
        const int t = idx / TILE, r = idx % TILE;
        const int row = (tile_m * GM + t / GN) * 16 * WM + r / (16 * WN), col = (tile_n * GN + t % GN) * 16 * WN + r % (16 * WN);
        if (row < M && col < N) store_result(e, row, col, s);
    }
}

// Tile shapes: BIG 64x64 by 2x2 wavefronts of 32x32; MID 32x32 and SMALL 16x16 by one output sub-tile, the wavefronts
// splitting k.  Rule: the largest tile that still gives half a chip of workgroups (128): the products here have few output
// tiles and the time of one is the time of its slowest workgroup, while a smaller tile reads its operands more often.  With 64 / 128 /
// 256 in its place, us: product 256 x 256, K = 3072 25.7 / 11.4 / 11.4, 512 x 256 26.9 / 26.7 / 23.4, 1024 x 256 97 / 27.7 / 27.7,
// 512 x 192, K = 384 5.5 / 6.0 / 6.0; backward pass of 3072 -> 256 at 32 rows 7.0 / 5.9 / 8.1, at 512 35.4 / 35.4 / 29.7, of 3136 -> 384 at
// 64 rows 9.5 / 9.5 / 13.3, at 128 21.1 / 15.3 / 15.3, at 256 25.1 / 24.8 / 30.1.
enum { BIG, MID, SMALL };
inline int tile_shape(int M, int N) {
    if ((long)ceil_div(M, 64) * ceil_div(N, 64) >= 128) return BIG;
    return (long)ceil_div(M, 32) * ceil_div(N, 32) >= 128 ? MID : SMALL;
}
__host__ __device__ constexpr int tile_edge(int shape) { return shape == BIG ? 64 : shape == MID ? 32 : 16; }

// The small tile fetches two k-chunks at a time.  With 1 / 2 / 3 / 4 / 6 of them, us: perceptron, batch 32, one worker 37.8 / 37.8 / 38.0 / 38.2 / 42.2; a push of the
// AlexNet-style network, batch 128, one worker 207.2 / 206.2 / 206.8 / 208.5 / 217.9, three convolutions, batch 37, 157.3 / 157.8 / 157.9 / 158.9 / 166.1.
template <int SHAPE, bool AV, bool BV>
__device__ __forceinline__ void shaped_tile(const Operand& a, const Operand& b, int M, int N, int K, int tile_m, int tile_n,
                                            const Epilogue& e, float* lds) {
    if constexpr (SHAPE == BIG) tile_product<2, 2, 2, 2, 1, AV, BV>(a, b, M, N, K, tile_m, tile_n, e, lds);
    else if constexpr (SHAPE == MID) tile_product<2, 2, 1, 1, 1, AV, BV>(a, b, M, N, K, tile_m, tile_n, e, lds);
    else tile_product<1, 1, 1, 1, 2, AV, BV>(a, b, M, N, K, tile_m, tile_n, e, lds);
}

// LDS (bytes) of a tile whose reduction is split over the wavefronts of `threads`
inline size_t tile_lds(int shape, int threads) {
    const int waves = threads / 64, kw = shape == BIG ? waves / 4 : waves;
    return kw > 1 ? sizeof(float) * waves * (shape == SMALL ? 256 : 1024) : 0;
}

// Arguments of the kernels from here on: pointers and numbers in front, which are in registers when a wavefront starts, and operands put together from them.  As
// structs they were a load from memory that every other one waited for: perceptron, batch 1, one worker 33.4 -> 31.4 us a push, batch 32 37.7 -> 36.0, AlexNet-style,
// batch 128, 207.8 -> 205.6.
// Layer z of the grid takes the reduction indices [z * k_per_layer, (z + 1) * k_per_layer) and writes its product to the
// z-th [M][N] slab of C (split-K with a second kernel; one layer otherwise).
template <int SHAPE, bool AV, bool BV>
__global__ __launch_bounds__(1024) void gemm_kernel(const float* __restrict__ a_p, const float* __restrict__ b_p, int M, int N, int K, int k_per_layer, long a_s,
                                                    long b_ks, long b_s, long a_ks, Epilogue e) {      // (numbers in front: they are there when a wavefront starts)
    extern __shared__ float lds[];
    Operand a{a_p, a_s, AV ? 1 : a_ks}, b{b_p, b_s, BV ? 1 : b_ks};
    const int k_lo = blockIdx.z * k_per_layer;
    a.p += (long)k_lo * a.ks; b.p += (long)k_lo * b.ks;
    e.C += (long)blockIdx.z * M * N;
    shaped_tile<SHAPE, AV, BV>(a, b, M, N, min(K - k_lo, k_per_layer), blockIdx.y, blockIdx.x, e, lds);
}

// Large products: a workgroup of four wavefronts owns a 64x64 tile and takes both operands through LDS, 16 reduction indices a stage,
// the next stage's loads in flight.  Each operand is read once per tile instead of twice, with lanes along whichever index is
// contiguous (K_FIRST: the reduction index), which is what counts once every compute unit has several tiles to work on and the
// caches no longer hold the operands.  Rule: from 1024 tiles, four to a compute unit.  Measured, A row-major / transposed / B
// transposed, this form against the one above: 256 tiles (1024^3) 55 / 55 / 53 against 36 / 39 / 49 us, 1024 tiles (2048^3)
// 201 / 202 / 193 against 241 / 258 / 249, 4096 tiles (4096 x 4096, K = 1024) 387 / 389 / 381 against 504 / 531 / 496.
constexpr int STAGED_TILES = 1024, STAGED_THREADS = 256;
template <bool A_K_FIRST, bool B_K_FIRST>
__global__ __launch_bounds__(STAGED_THREADS) void gemm_staged_kernel(Operand a, Operand b, Epilogue e, int M, int N, int K) {
    __shared__ __attribute__((aligned(16))) float As[2][64 * mma::LDK], Bs[2][64 * mma::LDK];        // [row of op(A) / column of op(B)][k]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    floatx4 acc[2][2];
    mma::zero(acc);
    float ra[4], rb[4];
    auto load = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int idx = tid + u * STAGED_THREADS;
            const int i = A_K_FIRST ? idx / 16 : idx % 64, ka = k0 + (A_K_FIRST ? idx % 16 : idx / 64);
            ra[u] = m0 + i < M && ka < K ? a.p[(long)(m0 + i) * a.s + (long)ka * a.ks] : 0.f;
            const int j = B_K_FIRST ? idx / 16 : idx % 64, kb = k0 + (B_K_FIRST ? idx % 16 : idx / 64);
            rb[u] = n0 + j < N && kb < K ? b.p[(long)(n0 + j) * b.s + (long)kb * b.ks] : 0.f;
        }
    };
    load(0);
    for (int k0 = 0, buf = 0; k0 < K; k0 += mma::KC, buf ^= 1) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int idx = tid + u * STAGED_THREADS;
            As[buf][A_K_FIRST ? idx / 16 * mma::LDK + idx % 16 : idx % 64 * mma::LDK + idx / 64] = ra[u];
            Bs[buf][B_K_FIRST ? idx / 16 * mma::LDK + idx % 16 : idx % 64 * mma::LDK + idx / 64] = rb[u];
        }
        __syncthreads();
        if (k0 + mma::KC < K) load(k0 + mma::KC);
        mma::chunk16<2, 2, false, true>(As[buf], mma::LDK, Bs[buf], mma::LDK, 32 * (wave >> 1), 32 * (wave & 1), acc, lane);
    }
    mma::drain();
    const int l16 = lane & 15, q = lane >> 4;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = m0 + 32 * (wave >> 1) + 16 * i + 4 * q + v, col = n0 + 32 * (wave & 1) + 16 * j + l16;
                if (row < M && col < N) store_result(e, row, col, acc[i][j][v]);
            }
}

// Threads of a workgroup: a wavefront is worth having for two k-chunks; up to 16 of them for the one-sub-tile shapes.
inline int tile_threads(int shape, int K) {
    const int chunks = ceil_div(K, mma::KC);
    if (shape == BIG) return 256;
    const int waves = chunks / 2 < 1 ? 1 : chunks / 2 > 16 ? 16 : chunks / 2;
    return 64 * waves;
}

inline bool vector_k(const Operand& o, int K) {
    return o.ks == 1 && o.s % 4 == 0 && K % 4 == 0 && (reinterpret_cast<uintptr_t>(o.p) & 15) == 0;
}

// out[slab][j] = sum over the rows i of the slab of X[i][j]: a workgroup owns 64 columns and one slab of rows
// (blockIdx.y), four row lanes each adding every fourth row of the slab in ascending order, eight loads in flight.
// Tall matrices take two passes (slab sums into scratch, then the sum of the slabs), short ones a single slab.
__device__ __forceinline__ void colsum_block(const float* __restrict__ X, float* __restrict__ out, long r0, long r1, int N, int col_block,
                                             float* lds) {
    float(*part)[64] = reinterpret_cast<float(*)[64]>(lds);       // [4][64]
    const int c = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int col = col_block * 64 + c;
    float s = 0.f;
    if (col < N) {
        long i = r0 + g;
        for (; i + 28 < r1; i += 32) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = X[(i + 4 * u) * N + col];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; i < r1; i += 4) s += X[i * N + col];
    }
    part[g][c] = s;
    __syncthreads();
    if (g == 0 && col < N) out[col] = (part[0][c] + part[1][c]) + (part[2][c] + part[3][c]);
}

__global__ __launch_bounds__(256) void colsum_kernel(const float* __restrict__ X, float* __restrict__ out, long M, int N,
                                                     long rows_per_slab) {
    __shared__ float lds[256];
    const long r0 = (long)blockIdx.y * rows_per_slab;
    colsum_block(X, out + (long)blockIdx.y * N, r0, r0 + rows_per_slab < M ? r0 + rows_per_slab : M, N, blockIdx.x, lds);
}

constexpr int COLSUM_SLABS = 256;

// C[i][j] = sum over the layers, in order, of partial[layer][i][j] (+ bias[j]) (ReLU)
__global__ __launch_bounds__(256) void splitk_sum_kernel(const float* __restrict__ partial, float* __restrict__ C, long ldc, int M,
                                                         int N, int layers, const float* __restrict__ bias, int relu) {
    const long e = (long)blockIdx.x * 256 + threadIdx.x;
    if (e >= (long)M * N) return;
    float s = 0.f;
    for (int l = 0; l < layers; ++l) s += partial[(long)l * M * N + e];
    const int col = (int)(e % N);
    if (bias) s += bias[col];
    if (relu) s = fmaxf(s, 0.f);
    C[(e / N) * ldc + col] = s;
}

int launch_gemm(hipStream_t s, const Operand& a, const Operand& b, const Epilogue& e, int M, int N, int K, int layers) {
    if (layers == 1 && (long)ceil_div(M, 64) * ceil_div(N, 64) >= STAGED_TILES) {
        const dim3 tiles(ceil_div(N, 64), ceil_div(M, 64)), threads(STAGED_THREADS);
#define GO(A, B) hipLaunchKernelGGL((gemm_staged_kernel<A, B>), tiles, threads, 0, s, a, b, e, M, N, K)
        if (a.ks == 1 && b.s == 1) GO(true, false); else if (a.ks == 1) GO(true, true); else if (b.s == 1) GO(false, false); else GO(false, true);
#undef GO
        return 1;
    }
    const int chunks = ceil_div(K, mma::KC);
    const int k_per_layer = ceil_div(chunks, layers) * mma::KC;
    const int shape = tile_shape(M, N), edge = tile_edge(shape), threads = tile_threads(shape, k_per_layer < K ? k_per_layer : K);
    const dim3 grid(ceil_div(N, edge), ceil_div(M, edge), ceil_div(K, k_per_layer));
    const bool av = vector_k(a, K), bv = vector_k(b, K);
    const size_t lds = tile_lds(shape, threads);
#define GO(S, AV, BV) hipLaunchKernelGGL((gemm_kernel<S, AV, BV>), grid, dim3(threads), lds, s, a.p, b.p, M, N, K, k_per_layer, a.s, b.ks, b.s, a.ks, e)
#define GO_V(S) do { if (av && bv) GO(S, true, true); else if (av) GO(S, true, false); else if (bv) GO(S, false, true); else GO(S, false, false); } while (0)
    if (shape == BIG) GO_V(BIG); else if (shape == MID) GO_V(MID); else GO_V(SMALL);
#undef GO_V
#undef GO
    return (int)grid.z;
}

// Backward pass of a fully connected layer y = x W + b in one launch: dW = x^T dy, db = column sums of dy, and (dx wanted)
// dx = dy W^T, masked by x > 0 if x is a post-ReLU activation; optionally also the mean of the mini-batch's losses.  The
// products do not depend on each other, so their tiles are workgroups of one grid; as kernels of their own (with the bias
// sums and the ReLU mask two more) each of them cost a dependent launch of 4 to 6 us.
struct FcBwd {
    float *dw, *db, *dx;
    int mask_dx;
    const float* row_loss; float* loss;
    int blocks_b;
};

constexpr int FC_THREADS = 256;

template <int SHW, int SHX, bool V>
__global__ __launch_bounds__(FC_THREADS) void fc_bwd_kernel(const float* __restrict__ x, const float* __restrict__ dy, const float* __restrict__ w, int m, int n_in,
                                                            int n_out, int blocks_x, int blocks_w, FcBwd f) {
    extern __shared__ float lds[];
    int b = blockIdx.x;
    if (b < blocks_x) {         // dx = dy W^T
        const int side = (n_in + tile_edge(SHX) - 1) / tile_edge(SHX);      // output tiles side by side
        shaped_tile<SHX, V, V>(Operand{dy, n_out, 1}, Operand{w, n_out, 1}, m, n_in, n_out, b / side, b % side, Epilogue{f.dx, n_in, nullptr, 0, f.mask_dx ? x : nullptr}, lds);
        return;
    }
    b -= blocks_x;
    if (b < blocks_w) {         // dW = x^T dy
        const int side = (n_out + tile_edge(SHW) - 1) / tile_edge(SHW);
        shaped_tile<SHW, false, false>(Operand{x, 1, n_in}, Operand{dy, 1, n_out}, n_in, n_out, m, b / side, b % side, Epilogue{f.dw, n_out, nullptr, 0, nullptr}, lds);
        return;
    }
    b -= blocks_w;
    if (b < f.blocks_b) {
        colsum_block(dy, f.db, 0, m, n_out, b, lds);
        return;
    }
    float s = 0.f;              // mean loss: a lane adds its samples in order, lanes by a tree
    for (int i = threadIdx.x; i < m; i += FC_THREADS) s += f.row_loss[i];
    lds[threadIdx.x] = s;
    __syncthreads();
    for (int h = FC_THREADS / 2; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) lds[threadIdx.x] += lds[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *f.loss = lds[0] / (float)m;
}

// Last layer and loss in one kernel: logits z = x W + b for 16 samples per workgroup (every class, at most 128), then the
// softmax of those rows from LDS: dz = (softmax(z) - onehot(y)) / m, row_loss[i] = logsumexp(z_i) - z_i[y_i].
// Eight wavefronts: class tiles side by side, the rest of them split the inputs.
constexpr int SX_WAVES = 8, SX_MAX_C = 128;
template <bool AV>
__global__ __launch_bounds__(64 * SX_WAVES) void fc_softmax_kernel(const float* __restrict__ x_p, const float* __restrict__ w_p, int m, int n_in, int C,
                                                                   const float* __restrict__ bias, const int32_t* __restrict__ label,
                                                                   float* __restrict__ z, float* __restrict__ dz, float* __restrict__ row_loss) {
    const Operand x{x_p, n_in, 1}, w{w_p, 1, C};
    __shared__ float part[SX_WAVES][16][17];
    __shared__ float Z[16][SX_MAX_C + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, q = lane >> 4;
    const int tiles = (C + 15) / 16, kw = SX_WAVES / tiles;        // tiles <= 8
    const int row0 = blockIdx.x * 16;
    if (wave < tiles * kw) {
        floatx4 acc[1][1];
        mma::zero(acc);
        wave_product<1, 1, 4, AV, false>(x, w, m, C, row0, 16 * (wave % tiles), n_in, wave / tiles, kw, acc, lane);
        mma::drain();
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave][4 * q + v][l16] = acc[0][0][v];
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < 16 * C; idx += 64 * SX_WAVES) {
        const int r = idx / C, c = idx - r * C;
        float s = 0.f;
        for (int p = 0; p < kw; ++p) s += part[p * tiles + c / 16][r][c % 16];
        s += bias[c];
        Z[r][c] = s;
        if (row0 + r < m) z[(long)(row0 + r) * C + c] = s;
    }
    __syncthreads();
    const float invm = 1.0f / (float)m;
    for (int r = wave; r < 16 && row0 + r < m; r += SX_WAVES) {
        const long i = row0 + r;
        float mx = -INFINITY;
        for (int j = lane; j < C; j += 64) mx = fmaxf(mx, Z[r][j]);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        float se = 0.f;
        for (int j = lane; j < C; j += 64) se += expf(Z[r][j] - mx);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) se += __shfl_xor(se, o);
        const int y = label[i];
        if (lane == 0) row_loss[i] = logf(se) + mx - Z[r][y];
        const float inv = 1.0f / se;
        for (int j = lane; j < C; j += 64) dz[i * C + j] = (expf(Z[r][j] - mx) * inv - (j == y ? 1.f : 0.f)) * invm;
    }
}

}  // namespace

extern "C" int dsspk_gemm(void* stream, const float* A, long a_rs, long a_cs, const float* B, long b_rs, long b_cs,
                          float* C, long ldc, int M, int N, int K, const float* bias, int relu) {
    if (!A || !B || !C || M < 1 || N < 1 || K < 1) return -1;
    launch_gemm((hipStream_t)stream, Operand{A, a_rs, a_cs}, Operand{B, b_cs, b_rs}, Epilogue{C, ldc, bias, relu, nullptr}, M, N, K, 1);
    return DSSPK_LAUNCH_RC();
}

// Split-K for callers who want more workgroups than a product has output tiles (the networks' layers do not: wavefronts of a
// workgroup split K without a second kernel).  Layers worth having: K of 1024 and more, fewer than 128 tiles of 64 x 64, at least 8
// k-chunks per layer, as many as give 384 workgroups of such tiles; the launch may cut the result into smaller ones (tile_shape).
extern "C" int dsspk_gemm_splitk_layers(int M, int N, int K) {
    if (M < 1 || N < 1 || K < 1) return 0;
    const int tiles = ceil_div(N, 64) * ceil_div(M, 64), chunks = ceil_div(K, mma::KC);
    if (tiles >= 128 || chunks < 64) return 1;
    const int want = ceil_div(384, tiles), most = chunks / 8;
    const int layers = want < most ? want : most;
    // as launched: the last layers may be empty once k_per_layer is rounded to whole chunks
    return ceil_div(K, ceil_div(chunks, layers) * mma::KC);
}

extern "C" int dsspk_gemm_splitk(void* stream, const float* A, long a_rs, long a_cs, const float* B, long b_rs, long b_cs,
                                 float* C, long ldc, int M, int N, int K, const float* bias, int relu, float* scratch, int layers) {
    if (!A || !B || !C || M < 1 || N < 1 || K < 1 || layers < 1) return -1;
    if (layers == 1) return dsspk_gemm(stream, A, a_rs, a_cs, B, b_rs, b_cs, C, ldc, M, N, K, bias, relu);
    if (!scratch) return -1;
    hipStream_t s = (hipStream_t)stream;
    const int launched = launch_gemm(s, Operand{A, a_rs, a_cs}, Operand{B, b_cs, b_rs}, Epilogue{scratch, N, nullptr, 0, nullptr}, M, N, K, layers);
    const long n = (long)M * N;
    hipLaunchKernelGGL(splitk_sum_kernel, dim3((unsigned)ceil_div(n, 256L)), dim3(256), 0, s, scratch, C, ldc, M, N, launched, bias, relu);
    return DSSPK_LAUNCH_RC();
}

extern "C" int dsspk_fc_bwd(void* stream, const float* x, const float* dy, const float* w, float* dw, float* db, float* dx, int mask_dx,
                            const float* row_loss, float* loss, int m, int n_in, int n_out) {
    if (!x || !dy || !dw || !db || (dx && !w) || (loss && !row_loss) || m < 1 || n_in < 1 || n_out < 1) return -1;
    const int shw = tile_shape(n_in, n_out), shx = tile_shape(m, n_in), ew = tile_edge(shw), ex = tile_edge(shx);
    const int blocks_w = ceil_div(n_out, ew) * ceil_div(n_in, ew), blocks_x = dx ? ceil_div(n_in, ex) * ceil_div(m, ex) : 0;
    const FcBwd f = {dw, db, dx, mask_dx, row_loss, loss, ceil_div(n_out, 64)};
    const int grid = blocks_x + blocks_w + f.blocks_b + (loss ? 1 : 0);
    const bool v = dx && vector_k(Operand{dy, n_out, 1}, n_out) && vector_k(Operand{w, n_out, 1}, n_out);
    size_t lds = tile_lds(shw, FC_THREADS), ldx = tile_lds(shx, FC_THREADS);
    if (lds < ldx) lds = ldx;
    if (lds < sizeof(float) * FC_THREADS) lds = sizeof(float) * FC_THREADS;
#define GO(W, X) do { if (v) hipLaunchKernelGGL((fc_bwd_kernel<W, X, true>), dim3(grid), dim3(FC_THREADS), lds, (hipStream_t)stream, x, dy, w, m, n_in, n_out, blocks_x, blocks_w, f); \
                      else hipLaunchKernelGGL((fc_bwd_kernel<W, X, false>), dim3(grid), dim3(FC_THREADS), lds, (hipStream_t)stream, x, dy, w, m, n_in, n_out, blocks_x, blocks_w, f); } while (0)
#define GO_X(W) do { if (shx == BIG) GO(W, BIG); else if (shx == MID) GO(W, MID); else GO(W, SMALL); } while (0)
    if (shw == BIG) GO_X(BIG); else if (shw == MID) GO_X(MID); else GO_X(SMALL);
#undef GO_X
#undef GO
    return DSSPK_LAUNCH_RC();
}

extern "C" int dsspk_fc_softmax_xent(void* stream, const float* x, const float* w, const float* bias, const int32_t* y, float* z,
                                     float* dz, float* row_loss, int m, int n_in, int C) {
    if (!x || !w || !bias || !y || !z || !dz || !row_loss || m < 1 || n_in < 1 || C < 1 || C > SX_MAX_C) return -1;
    const Operand a{x, n_in, 1};
    const dim3 grid(ceil_div(m, 16)), threads(64 * SX_WAVES);
    if (vector_k(a, n_in))
        hipLaunchKernelGGL((fc_softmax_kernel<true>), grid, threads, 0, (hipStream_t)stream, x, w, m, n_in, C, bias, y, z, dz, row_loss);
    else
        hipLaunchKernelGGL((fc_softmax_kernel<false>), grid, threads, 0, (hipStream_t)stream, x, w, m, n_in, C, bias, y, z, dz, row_loss);
    return DSSPK_LAUNCH_RC();
}

extern "C" size_t dsspk_colsum_scratch_floats(long M, int N) {
    return M > 1024 && N >= 1 ? (size_t)COLSUM_SLABS * N : 0;
}

extern "C" int dsspk_colsum(void* stream, const float* X, float* out, float* scratch, long M, int N) {
    if (!X || !out || M < 1 || N < 1) return -1;
    hipStream_t s = (hipStream_t)stream;
    if (dsspk_colsum_scratch_floats(M, N) == 0) {
        hipLaunchKernelGGL(colsum_kernel, dim3(ceil_div(N, 64), 1), dim3(256), 0, s, X, out, M, N, M);
        return DSSPK_LAUNCH_RC();
    }
    if (!scratch) return -1;
    const long rps = (M + COLSUM_SLABS - 1) / COLSUM_SLABS;
    const int slabs = ceil_div(M, rps);
    hipLaunchKernelGGL(colsum_kernel, dim3(ceil_div(N, 64), slabs), dim3(256), 0, s, X, scratch, M, N, rps);
    hipLaunchKernelGGL(colsum_kernel, dim3(ceil_div(N, 64), 1), dim3(256), 0, s, scratch, out, (long)slabs, N, (long)slabs);
    return DSSPK_LAUNCH_RC();
}

// ---- dsspk_colsum for callers that may not allocate: the slab sums go to device memory that is part of the library image
namespace {

constexpr int NOALLOC_MAX_N = DSSPK_COLSUM_NOALLOC_MAX_N;
constexpr int MAX_DEVICES = 64;

// One copy per GPU the library is loaded on, kept until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress: the device address it resolves to (per device) is what kernels and copies are given.
static __device__ __align__(256) float colsum_scratch[(size_t)COLSUM_SLABS * NOALLOC_MAX_N];

std::mutex scratch_mutex;
float* scratch_ptr[MAX_DEVICES];        // device address of colsum_scratch on each device, resolved on first use there

int resolve_scratch(float** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return DSSPK_NOALLOC_EHIP;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(colsum_scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return DSSPK_NOALLOC_EHIP;
        }
        scratch_ptr[dev] = static_cast<float*>(ptr);
    }
    *out = scratch_ptr[dev];
    return 0;
}

}  // namespace

extern "C" int dsspk_colsum_noalloc(void* stream, const float* X, float* out, long M, int N) {
    if (!X || !out || M < 1 || N < 1) return -1;
    if (N > NOALLOC_MAX_N) return DSSPK_NOALLOC_ETOOBIG;
    float* scratch = nullptr;
    if (int rc = resolve_scratch(&scratch)) return rc;
    // every slab row the second pass reads is written by the first pass of the same call, so nothing has to be cleared
    return dsspk_colsum(stream, X, out, scratch, M, N);
}
