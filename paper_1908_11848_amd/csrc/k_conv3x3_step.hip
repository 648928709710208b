// Launches of a residual network's step behind the C interface, so that the forms only a step takes (3x3 convolutions with filters converted ahead, a
// block's inner activation worked out again, the last stage's d-filter beside its d-input; both gradients of a stride-2 convolution; the end of the
// network) can be checked and timed on their own.
#include "common.hpp"
#include "conv3x3_layers.hpp"
#include "head.hpp"
#include "../../include/dssp_kernels.h"

namespace {
__global__ __launch_bounds__(FilterJob::THREADS) void filters_kernel(FilterJob job) { convert_filters(job, blockIdx.x); }
}  // namespace

extern "C" size_t dsspk_conv3x3_filter_bytes(int C) {
    return C == 16 || C == 32 || C == 64 ? 2 * filter3x3_uint4s(C) * sizeof(uint4) : 0;
}

extern "C" int dsspk_conv3x3_filters(void* stream, const float* w, void* planes, int C) {
    if (!w || !planes || dsspk_conv3x3_filter_bytes(C) == 0) return -1;
    FilterRun runs[3] = {};
    runs[C / 32].count = 1;
    const FilterJob job(w, (uint4*)planes, runs);
    hipLaunchKernelGGL(filters_kernel, dim3(job.blocks()), dim3(FilterJob::THREADS), 0, (hipStream_t)stream, job);
    return DSSPK_LAUNCH_RC();
}

extern "C" int dsspk_conv3x3_step_fwd(void* stream, int workgroups, const float* src, const float* records, int parts, const float* gamma,
                                      const float* beta, float eps, const float* shortcut, float* act_out, float* stats_out, const float* w,
                                      const void* planes, float* dst, float* records_out, int shortcut_half, int N, int H, int C) {
    if (!planes) return -1;
    const Filter3x3 f(w, (const uint4*)planes);
    hipStream_t s = (hipStream_t)stream;
    if (workgroups == DSSPK_CONV3X3_SMALL || workgroups == DSSPK_CONV3X3_LARGE)
        return (workgroups == DSSPK_CONV3X3_SMALL ? conv3x3_small_fwd : conv3x3_large_fwd)(s, src, records, parts, gamma, beta, eps, shortcut, act_out,
                                                                                          stats_out, f, dst, records_out, shortcut_half, N, H, C);
    if (workgroups != DSSPK_CONV3X3_MEDIUM || !src || !w || !dst || !records_out || dst == src || N < 1 || conv3x3_tiled_stat_parts(N, H, C) == 0) return -1;
    if (shortcut_half && (!shortcut || C <= 16)) return -1;
    if (!records) return parts || shortcut ? -1 : conv3x3_tiled(s, src, f, nullptr, dst, records_out, N, H, C, false);
    if (!gamma || !beta || !act_out || !stats_out || act_out == src || act_out == dst || records == records_out) return -1;
    return conv3x3_tiled_prebn(s, src, records, parts, gamma, beta, eps, shortcut, shortcut_half != 0, act_out, stats_out, f, dst, records_out, N, H, C);
}

extern "C" int dsspk_conv3x3_step_bwd(void* stream, int workgroups, const float* dz, const float* xc, const float* stats, const float* gamma,
                                      const float* totals, const float* in_records, int parts, float* dgamma, float* dbeta, float* dx, float* partial,
                                      const float* w, const void* planes, const float* add, float* out, const float* x_in, const float* xc_post,
                                      const float* stats_post, const float* gamma_post, const float* beta_post, float* records,
                                      const float* red_partial, float* red_dw, int red_E, int red_chunks, int red_quads, int N, int H, int C) {
    if (!planes || !gamma_post != !beta_post || (red_quads && red_chunks > 64)) return -1;
    const Filter3x3 f(w, (const uint4*)planes + filter3x3_uint4s(C));
    hipStream_t s = (hipStream_t)stream;
    if (workgroups == DSSPK_CONV3X3_SMALL || workgroups == DSSPK_CONV3X3_LARGE) {
        if (totals) return -1;
        return (workgroups == DSSPK_CONV3X3_SMALL ? conv3x3_small_bwd : conv3x3_large_bwd)(
            s, dz, xc, stats, gamma, in_records, parts, dgamma, dbeta, dx, partial, f, add, out, x_in, xc_post, stats_post, records,
            jobs::Partials{red_partial, red_dw, red_E, red_chunks, red_quads != 0}, N, H, C, gamma_post, beta_post);
    }
    if (workgroups != DSSPK_CONV3X3_MEDIUM || red_quads || N < 1 || conv3x3_tiled_stat_parts(N, H, C) == 0) return -1;
    if (!dz || !xc || !stats || !gamma || !totals || in_records || !w || !out || out == dz || !x_in || !xc_post || !stats_post || !records) return -1;
    if (C == 64 ? !dx || partial || dx == dz || dx == out : dx || !partial || partial == red_partial) return -1;
    if (red_partial && (!red_dw || red_E < 4 || red_E % 4 || red_chunks < 1)) return -1;
    if (C == 64)
        return conv3x3_tiled_dgrad_bn(s, dz, xc, stats, gamma, totals, nullptr, 0, nullptr, nullptr, dx, f, add, out, x_in, xc_post, stats_post, records,
                                      red_partial, red_dw, red_E, red_chunks, N, H, C, gamma_post, beta_post);
    return conv3x3_tiled_dgrad_bn_wgrad(s, dz, xc, stats, gamma, totals, nullptr, 0, nullptr, nullptr, f, add, out, xc_post, stats_post, records, x_in,
                                        partial, red_partial, red_dw, red_E, red_chunks, N, H, C, gamma_post, beta_post);
}

extern "C" int dsspk_stride2_step_records(int N, int H, int Cin) { return conv_stride2_bwd_records(N, H, Cin); }

extern "C" int dsspk_stride2_step_bwd(void* stream, const float* dy, const float* w, const float* shortcut, float* dx, float* partial, const float* x_in,
                                      const float* xc_post, const float* stats_post, float* records, int N, int H, int Cin, int* chunks_out) {
    if (!chunks_out || dx == dy || dx == x_in || dx == xc_post || partial == dx || records == partial) return -1;
    return conv_stride2_bwd((hipStream_t)stream, dy, w, shortcut, dx, partial, BehindBn{x_in, xc_post, stats_post, records}, N, H, Cin, chunks_out);
}

extern "C" int dsspk_head_step_takes(int N, int parts, int classes) { return N >= 1 && resnet_head_takes(N, parts, classes); }

extern "C" int dsspk_head_step(void* stream, const float* x, const float* records, int parts, const float* gamma_beta, const float* shortcut,
                               int shortcut_half, const float* w_bias, const int32_t* label, float eps, float* out, float* stats, float* pooled, float* logits,
                               float* dlogits, float* row_loss, float* dz, float* records_out, int N, int classes) {
    if (!dsspk_head_step_takes(N, parts, classes)) return -1;
    if (!label || !out || !stats || !pooled || !logits || !dlogits || !row_loss || !dz || !records_out || dz == out) return -1;
    const HeadArgs a = {out, stats, label, pooled, logits, dlogits, row_loss, dz, records_out, eps, 1.f / (float)N, (int)((long)N * 64 / parts), classes};
    return resnet_head((hipStream_t)stream, x, records, parts, gamma_beta, shortcut, shortcut_half != 0, w_bias, N, a);
}
