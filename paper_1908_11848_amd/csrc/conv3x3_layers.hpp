// The launchers of the 3x3 kernels (conv3x3.hpp) inside the library: those of include/dssp_kernels.h, with a filter that may have been
// converted already.
#pragma once
#include "conv3x3_filter.hpp"
#include "jobs.hpp"

// k_conv.hip: a residual network's first layer (3 -> 16 channels on 32x32), which carries the conversion of the filters behind it.  records as of
// dsspk_conv_fwd_records, or NULL.
int conv_stem(hipStream_t s, const float* x, const float* w, float* y, float* records, int N, FilterJob job);

// k_conv.hip: a residual network's stride-2 3x3 convolution (16 -> 32 channels on 32x32, 32 -> 64 on 16x16; at most 32 images): dsspk_conv_bwd_data_shortcut and the
// first stage of its d-filter, with the backward pass of the ReLU and batch norm in front begun: dx is masked by mask > 0 (the convolution's input, that
// norm's output behind the ReLU) and the sums of dx and dx * xhat, xhat of xc and stats, are left as records.  ..records: how many; 0: shape not taken.
struct BehindBn { const float *mask, *xc, *stats; float* records; };
int conv_stride2_bwd_records(int N, int H, int Cin);
int conv_stride2_bwd(hipStream_t s, const float* dy, const float* w, const float* shortcut, float* dx, float* partial, const BehindBn& behind, int N, int H, int Cin,
                     int* chunks_out);

int wgrad_reduce_many(hipStream_t s, int n, const jobs::Partials* waiting);

// k_conv3x3.hip; -2 = shape not covered.
int conv3x3_tiled(hipStream_t s, const float* src, const Filter3x3& w, const float* add, float* dst, float* bn_partial,
                   int N, int HW, int C, bool transposed);
int conv3x3_tiled_stat_parts(int N, int HW, int C);
int conv3x3_tiled_dgrad_post(hipStream_t s, const float* dy, const float* w, const float* add, float* dz,
                              const float* mask_src, const float* xc, const float* stats, float* records, int N, int HW, int C);
int conv3x3_tiled_prebn(hipStream_t s, const float* src, const float* records, int in_parts, const float* gamma,
                         const float* beta, float eps, const float* shortcut, bool half, float* act_out, float* stats_out,
                         const Filter3x3& w, float* dst, float* bn_partial, int N, int HW, int C);
int wgrad3x3_tiled_parts(int N, int HW, int C);
int wgrad3x3_tiled(hipStream_t s, const float* x, const float* dy, float* partial, int N, int HW, int C, const jobs::TotalsJob& tj);
// The batch norm's sums: totals, or (totals null) parts records to add up, dgamma and dbeta stored from them.
bool conv3x3_records_inline(int parts, int C);
int conv3x3_tiled_dgrad_bn(hipStream_t s, const float* dz, const float* xc, const float* stats, const float* gamma,
                            const float* totals, const float* in_records, int parts, float* dgamma, float* dbeta, float* dx_out,
                            const Filter3x3& w, const float* add, float* out,
                            const float* mask_src, const float* xc_post, const float* stats_post, float* records,
                            const float* red_partial, float* red_dw, int red_E, int red_chunks, int N, int HW, int C,
                            const float* gamma_post = nullptr, const float* beta_post = nullptr);
int conv3x3_tiled_dgrad_bn_wgrad(hipStream_t s, const float* dz, const float* xc, const float* stats, const float* gamma,
                                  const float* totals, const float* in_records, int parts, float* dgamma, float* dbeta,
                                  const Filter3x3& w, const float* add, float* out,
                                  const float* xc_post, const float* stats_post, float* records,
                                  const float* x_in, float* partial, const float* red_partial, float* red_dw, int red_E,
                                  int red_chunks, int N, int HW, int C, const float* gamma_post = nullptr, const float* beta_post = nullptr);

// k_conv3x3_large.hip, k_conv3x3_small.hip: dsspk_conv3x3_large_* and dsspk_conv3x3_small_*.  small_bwd with converted filters takes `partial` for 64
// channels too: one partial result an image, to be reduced as Partials::quads.  gamma_post, beta_post:
// of the batch norm of xc_post, if x_in is ReLU(BN(xc_post)) with nothing added (else NULL).
#define CONV3X3_FORM_LAUNCHERS(NAME)                                                                                                          \
    int conv3x3_##NAME##_fwd(void* stream, const float* src, const float* records, int parts, const float* gamma, const float* beta,         \
                             float eps, const float* shortcut, float* act_out, float* stats_out, const Filter3x3& w, float* dst,              \
                             float* records_out, int shortcut_half, int N, int H, int C);                                                     \
    int conv3x3_##NAME##_bwd(void* stream, const float* dz, const float* xc, const float* stats, const float* gamma,                         \
                             const float* in_records, int parts, float* dgamma, float* dbeta, float* dx, float* partial,                      \
                             const Filter3x3& w, const float* add, float* out, const float* x_in, const float* xc_post,                       \
                             const float* stats_post, float* records, const jobs::Partials& red, int N, int H, int C, const float* gamma_post,  \
                             const float* beta_post);
CONV3X3_FORM_LAUNCHERS(large)
CONV3X3_FORM_LAUNCHERS(small)
int conv3x3_small_records(int C);            // records of a tensor of C channels that a small workgroup adds up, at most
