// The full set of launches of the 3x3 kernels of conv3x3.hpp with one choice of workgroup (`F`: wavefronts, rows of a band, channel splits,
// images at most), behind dsspk_conv3x3_large_* and dsspk_conv3x3_small_*.
#pragma once
#include "conv3x3.hpp"
#include "conv3x3_layers.hpp"

namespace {

template <class F> int form_parts(int N, int H, int C) {
    if (N < 1 || N > F::IMAGES) return 0;
    return C == 16 && H == 32 ? N * (32 / F::R16) : C == 32 && H == 16 ? N * (16 / F::R32) : C == 64 && H == 8 ? N : 0;
}

// Records that a workgroup adds up itself, at most.
template <class F> int form_records(int C) {
    return C == 16   ? inline_records<16, F::WAVES, F::TILES>()
           : C == 32 ? inline_records<32, F::WAVES, F::TILES>()
                     : inline_records<64, F::WAVES, F::TILES>();
}
template <class F> bool form_merges(int parts, int C) { return parts >= 1 && parts <= form_records<F>(C); }

template <class F, int PRE>
int form_launch(hipStream_t s, const float* src, const Filter3x3& w, float* dst, float* records_out, int N, int C, const PreBn& pre) {
    if (C == 16) return launch<16, 32, F::R16, 1, F::WAVES, false, PRE>(s, src, w, nullptr, dst, records_out, N, pre);
    if (C == 32) return launch<32, 16, F::R32, 1, F::WAVES, false, PRE>(s, src, w, nullptr, dst, records_out, N, pre);
    return launch<64, 8, 8, F::SPLIT64, F::WAVES, false, PRE>(s, src, w, nullptr, dst, records_out, N, pre);
}

template <class F>
int form_fwd(void* stream, const float* src, const float* records, int parts, const float* gamma, const float* beta, float eps,
             const float* shortcut, float* act_out, float* stats_out, const Filter3x3& w, float* dst, float* records_out, int shortcut_half, int N,
             int H, int C) {
    if (!src || !w.w || !dst || !records_out || dst == src || form_parts<F>(N, H, C) == 0) return -1;
    if (shortcut_half && (!shortcut || C <= 16)) return -1;
    PreBn pre{};
    pre.half = shortcut_half != 0;
    if (!records) {
        if (parts || shortcut) return -1;
        return form_launch<F, 0>((hipStream_t)stream, src, w, dst, records_out, N, C, pre);
    }
    const long M = (long)N * H * H;
    if (!gamma || !beta || !act_out || !stats_out || act_out == src || act_out == dst || records == records_out || !form_merges<F>(parts, C) || M % parts) return -1;
    pre.records = records;
    pre.M = M;
    pre.parts = parts;
    pre.rows = M / parts;
    pre.gamma = gamma; pre.beta = beta; pre.eps = eps;
    pre.shortcut = shortcut; pre.act_out = act_out; pre.stats_out = stats_out;
    pre.merge = true;
    return shortcut ? form_launch<F, 2>((hipStream_t)stream, src, w, dst, records_out, N, C, pre)
                    : form_launch<F, 1>((hipStream_t)stream, src, w, dst, records_out, N, C, pre);
}

template <class F>
int form_bwd(void* stream, const float* dz, const float* xc, const float* stats, const float* gamma, const float* in_records, int parts,
             float* dgamma, float* dbeta, float* dx, float* partial, const Filter3x3& w, const float* add, float* out, const float* x_in,
             const float* xc_post, const float* stats_post, float* records, const jobs::Partials& red, int N, int H, int C,
             const float* gamma_post = nullptr, const float* beta_post = nullptr) {
    if (!dz || !xc || !stats || !gamma || !in_records || !dgamma || !dbeta || !w.w || !out || !x_in || !xc_post || !stats_post || !records) return -1;
    if (form_parts<F>(N, H, C) == 0 || !form_merges<F>(parts, C) || in_records == records || out == dz) return -1;
    // 64 channels: dx for a d-filter kernel of its own or, in a network's step with small workgroups, the partial filter gradients (one an image)
    const bool fused = C < 64 || (F::SPLIT64 == 4 && w.planes && partial);
    if (fused ? dx || !partial || partial == red.partial : !dx || partial || dx == dz || dx == out) return -1;
    if (red.partial && (!red.dw || red.E < 4 || red.E % 4 || red.chunks < 1)) return -1;
    BwdBn bwd;
    bwd.xc = xc; bwd.stats = stats; bwd.gamma = gamma; bwd.totals = nullptr; bwd.records = in_records; bwd.parts = parts;
    bwd.dgamma = dgamma; bwd.dbeta = dbeta; bwd.inv_m = 1.0f / (float)((long)N * H * H); bwd.dx_out = dx;
    PostBn post{};
    post.mask_src = x_in; post.xc = xc_post; post.stats = stats_post; post.records = records; post.gamma = gamma_post; post.beta = beta_post;
    const jobs::ReduceJob rj = reduce_job(red, 64 * F::WAVES);
    WgradFused wg;
    wg.x_in = x_in; wg.partial = partial;
    hipStream_t s = (hipStream_t)stream;
    if (C == 16) return launch<16, 32, F::R16, 1, F::WAVES, true, 3, true, true>(s, dz, w, add, out, nullptr, N, PreBn{}, post, bwd, rj, wg);
    if (C == 32) return launch<32, 16, F::R32, 1, F::WAVES, true, 3, true, true>(s, dz, w, add, out, nullptr, N, PreBn{}, post, bwd, rj, wg);
    if constexpr (F::SPLIT64 == 4)
        return fused ? gamma_post ? launch_form<true, 64, 8, 8, 4, F::WAVES, true, 3, true, true, true>(s, dz, w, add, out, nullptr, N, PreBn{}, post, bwd, rj, wg)
                                  : launch_form<true, 64, 8, 8, 4, F::WAVES, true, 3, true, true>(s, dz, w, add, out, nullptr, N, PreBn{}, post, bwd, rj, wg)
                     : launch_form<false, 64, 8, 8, 4, F::WAVES, true, 3, true, false>(s, dz, w, add, out, nullptr, N, PreBn{}, post, bwd, rj, wg);
    else
        return launch<64, 8, 8, F::SPLIT64, F::WAVES, true, 3, true>(s, dz, w, add, out, nullptr, N, PreBn{}, post, bwd, rj);
}

}  // namespace

#define DSSPK_CONV3X3_FORM(NAME, F)                                                                                                                \
    int conv3x3_##NAME##_fwd(void* stream, const float* src, const float* records, int parts, const float* gamma, const float* beta,              \
                             float eps, const float* shortcut, float* act_out, float* stats_out, const Filter3x3& w, float* dst,                   \
                             float* records_out, int shortcut_half, int N, int H, int C) {                                                         \
        return form_fwd<F>(stream, src, records, parts, gamma, beta, eps, shortcut, act_out, stats_out, w, dst, records_out, shortcut_half, N, H, \
                           C);                                                                                                                     \
    }                                                                                                                                              \
    int conv3x3_##NAME##_bwd(void* stream, const float* dz, const float* xc, const float* stats, const float* gamma,                              \
                             const float* in_records, int parts, float* dgamma, float* dbeta, float* dx, float* partial,                           \
                             const Filter3x3& w, const float* add, float* out, const float* x_in, const float* xc_post,                            \
                             const float* stats_post, float* records, const jobs::Partials& red, int N, int H, int C, const float* gamma_post,     \
                             const float* beta_post) {                                                                                             \
        return form_bwd<F>(stream, dz, xc, stats, gamma, in_records, parts, dgamma, dbeta, dx, partial, w, add, out, x_in, xc_post, stats_post,   \
                           records, red, N, H, C, gamma_post, beta_post);                                                                          \
    }                                                                                                                                              \
    extern "C" int dsspk_conv3x3_##NAME##_parts(int N, int H, int C) { return form_parts<F>(N, H, C); }                                            \
    extern "C" int dsspk_conv3x3_##NAME##_fwd(void* stream, const float* src, const float* records, int parts, const float* gamma,                \
                                              const float* beta, float eps, const float* shortcut, float* act_out, float* stats_out,              \
                                              const float* w, float* dst, float* records_out, int shortcut_half, int N, int H, int C) {           \
        return conv3x3_##NAME##_fwd(stream, src, records, parts, gamma, beta, eps, shortcut, act_out, stats_out, w, dst, records_out,             \
                                    shortcut_half, N, H, C);                                                                                       \
    }                                                                                                                                              \
    extern "C" int dsspk_conv3x3_##NAME##_bwd(void* stream, const float* dz, const float* xc, const float* stats, const float* gamma,             \
                                              const float* in_records, int parts, float* dgamma, float* dbeta, float* dx, float* partial,         \
                                              const float* w, const float* add, float* out, const float* x_in, const float* xc_post,              \
                                              const float* stats_post, float* records, const float* red_partial, float* red_dw, int red_E,        \
                                              int red_chunks, int N, int H, int C) {                                                               \
        return conv3x3_##NAME##_bwd(stream, dz, xc, stats, gamma, in_records, parts, dgamma, dbeta, dx, partial, w, add, out, x_in, xc_post,      \
                                    stats_post, records, jobs::Partials{red_partial, red_dw, red_E, red_chunks, false}, N, H, C, nullptr, nullptr); \
    }
