// The networks of the workloads as fixed launch sequences (internal, see model.hpp), and the
// host-only queries about their parameter vector and workspace.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "../../include/dssp.h"
#include "../../include/dssp_kernels.h"
#include "conv3x3_layers.hpp"
#include "conv_split_layers.hpp"
#include "head.hpp"
#include "model.hpp"

namespace dssp_model {

namespace {

struct Seg { int32_t kind; int64_t size, fan_in; };
enum { KW_ = 0, KB_ = 1, KG_ = 2, KBETA_ = 3 };

bool is_resnet(int id) { return id >= 8 && (id - 2) % 6 == 0; }

struct ResBlock {
    int H, cin, cout, stride;              // H: input height = width
    int64_t w1, g1, b1, w2, g2, b2;        // offsets into the flat parameter vector (floats)
    size_t c1, a1, c2, out, st1, st2;      // offsets into the worker's workspace slice (bytes)
    size_t f1, f2;                         // the converted filters of the two convolutions (conv3x3_filter.hpp), f1 of a stride-1 block
};

// Bump allocator over one worker's slice of the workspace (256-byte granules).
struct Arena {
    size_t off = 0;
    size_t take(size_t bytes) { const size_t o = off; off += (bytes + 255) / 256 * 256; return o; }
    size_t floats(size_t n) { return take(n * sizeof(float)); }
};

}  // namespace

// d-filter partial sums wait in scratch buffers until a later kernel carries their reduction: at most four at a time (one per regular
// layer in a row, one more per stage boundary, the stem's), and one is being written.
constexpr int WG_SCRATCH = 5;
static_assert(WG_SCRATCH - 1 <= DSSPK_WGRAD_REDUCE_MAX, "what waits is one launch");

struct Plan {
    int model_id = 0, m = 0, n_classes = 0, K = 0;
    char* ws = nullptr;
    size_t per_worker = 0;
    std::vector<Seg> segs;
    int64_t n_params = 0;
    // tensors tests may look at: (what, byte offset in the worker slice, element count)
    struct Tens { int what; size_t off; int64_t count; };
    std::vector<Tens> tens;

    // common tail
    size_t logits = 0, dlogits = 0, row_loss = 0, wg_scratch = 0, wg_more[WG_SCRATCH - 1] = {}, bn_scratch = 0, bn_scratch2 = 0, tot_a = 0, tot_b = 0;
    // MLP
    size_t mlp_a1 = 0, mlp_da1 = 0;
    // AlexNet-style
    size_t ax_a1 = 0, ax_p1 = 0, ax_arg1 = 0, ax_a2 = 0, ax_p2 = 0, ax_arg2 = 0, ax_a3 = 0, ax_a4 = 0;
    size_t ax_da4 = 0, ax_da3 = 0, ax_dp2 = 0, ax_da2 = 0, ax_dp1 = 0;
    size_t ax_c3 = 0, ax_dc3 = 0;     // three-convolution variant: conv3 output (post-ReLU) and its gradient
    struct WideConv { size_t fwd = 0, bwd = 0, partial = 0; } wide2, wide3;      // the convolutions behind the first one: filter planes, partial filter gradients
    // ResNet
    std::vector<ResBlock> blocks;
    int64_t stem_w = 0, stem_g = 0, stem_b = 0, fc_w = 0, fc_b = 0;
    size_t filters = 0;
    FilterRun filter_runs[3] = {};
    size_t stem_c = 0, stem_a = 0, stem_st = 0, pooled = 0, dpooled = 0, G[3] = {0, 0, 0};

    void seg(int kind, int64_t size, int64_t fan_in) { segs.push_back({kind, size, fan_in}); n_params += size; }
    int64_t conv_seg(int k, int cin, int cout, bool bias) {
        const int64_t o = n_params;
        seg(KW_, (int64_t)k * k * cin * cout, (int64_t)k * k * cin);
        if (bias) seg(KB_, cout, 0);
        return o;
    }
    int64_t fc_seg(int in, int out) {
        const int64_t o = n_params;
        seg(KW_, (int64_t)in * out, in);
        seg(KB_, out, 0);
        return o;
    }
    int64_t bn_seg(int c) {
        const int64_t o = n_params;
        seg(KG_, c, 0);
        seg(KBETA_, c, 0);
        return o;
    }

    bool build(int id, int batch, int classes) {
        model_id = id; m = batch; n_classes = classes;
        Arena a;
        size_t wg = 0, bn = 0;
        auto wg_need = [&](int N, int H, int Cin, int Cout, int k, int s, int p) {
            const size_t f = dsspk_conv_wgrad_scratch_floats(N, H, H, Cin, Cout, k, k, s, p);
            if (f > wg) wg = f;
            if (k == 3 && s == 1 && Cin == Cout) wg = std::max(wg, (size_t)dsspk_conv3x3_small_parts(N, H, Cin) * 9 * Cin * Cout);
        };
        // wide stride-1 layer (dsspk_conv_split_*): room for its filter planes and the partial sums of its d-filter pass, which wait for the end of
        // the step
        auto wide_conv = [&](WideConv& c, int H, int k, int p) {
            c.partial = a.floats(dsspk_conv_split_wgrad_scratch_floats(m, H, H, 64, 64, k, p));
            c.fwd = a.take(dsspk_conv_split_filter_bytes(64, 64, k));
            c.bwd = a.take(dsspk_conv_split_filter_bytes(64, 64, k));
        };
        auto bn_need = [&](long M, int C) { const size_t f = dsspk_bn_scratch_floats(M, C); if (f > bn) bn = f; };
        if (id == DSSP_MODEL_MLP) {
            fc_seg(3072, 256);
            fc_seg(256, classes);
            mlp_a1 = a.floats((size_t)m * 256);
            mlp_da1 = a.floats((size_t)m * 256);
            tens.push_back({0, mlp_a1, (int64_t)m * 256});
        } else if (id == DSSP_MODEL_ALEXNET_DS) {
            conv_seg(5, 3, 64, true);
            conv_seg(5, 64, 64, true);
            fc_seg(7 * 7 * 64, 384);
            fc_seg(384, 192);
            fc_seg(192, classes);
            const size_t s32 = (size_t)m * 32 * 32 * 64, s15 = (size_t)m * 15 * 15 * 64, s7 = (size_t)m * 7 * 7 * 64;
            ax_a1 = a.floats(s32); ax_p1 = a.floats(s15); ax_arg1 = a.take(s15);
            ax_a2 = a.floats(s15); ax_p2 = a.floats(s7); ax_arg2 = a.take(s7);
            ax_a3 = a.floats((size_t)m * 384); ax_a4 = a.floats((size_t)m * 192);
            ax_da4 = a.floats((size_t)m * 192); ax_da3 = a.floats((size_t)m * 384); ax_dp2 = a.floats(s7);
            ax_da2 = a.floats(s15); ax_dp1 = a.floats(s15);
            wg = dsspk_conv_first_scratch_floats(m);
            wide_conv(wide2, 15, 5, 2);
            tens.push_back({0, ax_a1, (int64_t)s32}); tens.push_back({0, ax_a2, (int64_t)s15});
            tens.push_back({0, ax_a3, (int64_t)m * 384}); tens.push_back({0, ax_a4, (int64_t)m * 192});
            tens.push_back({1, ax_arg1, (int64_t)s15}); tens.push_back({1, ax_arg2, (int64_t)s7});
        } else if (id == DSSP_MODEL_ALEXNET_3C) {
            conv_seg(5, 3, 64, true);
            conv_seg(5, 64, 64, true);
            conv_seg(3, 64, 64, true);
            fc_seg(7 * 7 * 64, 384);
            fc_seg(384, classes);
            const size_t s32 = (size_t)m * 32 * 32 * 64, s15 = (size_t)m * 15 * 15 * 64, s7 = (size_t)m * 7 * 7 * 64, s7c = s7;
            ax_a1 = a.floats(s32); ax_p1 = a.floats(s15); ax_arg1 = a.take(s15);
            ax_a2 = a.floats(s15); ax_p2 = a.floats(s7); ax_arg2 = a.take(s7);
            ax_c3 = a.floats(s7c); ax_a3 = a.floats((size_t)m * 384);
            ax_da3 = a.floats((size_t)m * 384); ax_dc3 = a.floats(s7c); ax_dp2 = a.floats(s7);
            ax_da2 = a.floats(s15); ax_dp1 = a.floats(s15);
            wg = dsspk_conv_first_scratch_floats(m);
            wide_conv(wide2, 15, 5, 2);
            wide_conv(wide3, 7, 3, 1);
            tens.push_back({0, ax_a1, (int64_t)s32}); tens.push_back({0, ax_a2, (int64_t)s15});
            tens.push_back({0, ax_c3, (int64_t)s7c}); tens.push_back({0, ax_a3, (int64_t)m * 384});
            tens.push_back({1, ax_arg1, (int64_t)s15}); tens.push_back({1, ax_arg2, (int64_t)s7});
        } else if (is_resnet(id)) {
            const int n = (id - 2) / 6;
            stem_w = conv_seg(3, 3, 16, false);
            stem_g = bn_seg(16); stem_b = stem_g + 16;
            const size_t s0 = (size_t)m * 32 * 32 * 16;
            stem_c = a.floats(s0); stem_a = a.floats(s0); stem_st = a.floats(32);
            tens.push_back({0, stem_a, (int64_t)s0});
            wg_need(m, 32, 3, 16, 3, 1, 1);
            bn_need((long)m * 32 * 32, 16);
            int cin = 16, H = 32;
            const int widths[3] = {16, 32, 64};
            for (int st = 0; st < 3; ++st)
                for (int b = 0; b < n; ++b) {
                    ResBlock B;
                    B.cin = cin; B.cout = widths[st]; B.stride = (st > 0 && b == 0) ? 2 : 1; B.H = H;
                    const int Ho = H / B.stride;
                    B.w1 = conv_seg(3, B.cin, B.cout, false); B.g1 = bn_seg(B.cout); B.b1 = B.g1 + B.cout;
                    B.w2 = conv_seg(3, B.cout, B.cout, false); B.g2 = bn_seg(B.cout); B.b2 = B.g2 + B.cout;
                    const size_t sz = (size_t)m * Ho * Ho * B.cout;
                    B.c1 = a.floats(sz); B.a1 = a.floats(sz); B.c2 = a.floats(sz); B.out = a.floats(sz);
                    B.st1 = a.floats(2 * B.cout); B.st2 = a.floats(2 * B.cout);
                    tens.push_back({0, B.a1, (int64_t)sz}); tens.push_back({0, B.out, (int64_t)sz});
                    wg_need(m, H, B.cin, B.cout, 3, B.stride, 1);
                    wg_need(m, Ho, B.cout, B.cout, 3, 1, 1);
                    bn_need((long)m * Ho * Ho, B.cout);
                    blocks.push_back(B);
                    cin = B.cout; H = Ho;
                }
            fc_w = fc_seg(64, classes); fc_b = fc_w + 64 * (int64_t)classes;
            pooled = a.floats((size_t)m * 64); dpooled = a.floats((size_t)m * 64);
            for (int i = 0; i < 3; ++i) G[i] = a.floats(s0);
            // A stage's filters of stride-1 convolutions are evenly spaced in the parameters: all of the first stage's, from the second
            // convolution on in the others.
            size_t uint4s = 0;
            for (int st = 0; st < 3; ++st) {
                const int C = widths[st], per = 9 * C * C + 2 * C;
                filter_runs[st] = {st ? blocks[st * n].w2 : blocks[0].w1, st ? 2 * n - 1 : 2 * n, per};
                for (int i = 0; i < filter_runs[st].count; ++i, uint4s += 2 * filter3x3_uint4s(C)) {
                    const int conv = st ? i + 1 : i;
                    ResBlock& B = blocks[st * n + conv / 2];
                    (conv % 2 ? B.f2 : B.f1) = uint4s;
                }
            }
            filters = a.take(uint4s * sizeof(uint4));
        } else {
            return false;
        }
        logits = a.floats((size_t)m * classes);
        dlogits = a.floats((size_t)m * classes);
        tens.push_back({2, logits, (int64_t)m * classes});
        row_loss = a.floats((size_t)m);
        wg_scratch = a.floats(wg ? wg : 1);
        for (size_t& o : wg_more) o = a.floats(is_resnet(id) && wg ? wg : 1);
        bn_scratch = a.floats(bn ? bn : 1);
        bn_scratch2 = a.floats(bn ? bn : 1);
        tot_a = a.floats(128); tot_b = a.floats(128);          // batch-norm backward sums (2 x 64 channels at most)
        per_worker = a.off;
        return true;
    }
};

namespace {

#define RUN(call)                                                        \
    do {                                                                 \
        const int rc_ = (call);                                          \
        if (rc_) { err = #call; return rc_; }                            \
    } while (0)

// Last fully connected layer (input a [m][n_in], weights at w + fw, biases at w + fb), softmax cross-entropy and the
// backward pass of that layer: logits, dlogits, gradients of fw / fb, the mini-batch's loss, and d_in (masked by a > 0 if
// mask), the gradient in front of a.
int last_layer(Plan* P, char* ws, void* s, const float* a, int n_in, const int32_t* y, const float* w, float* g, int64_t fw, int64_t fb,
               float* d_in, int mask, float* loss, std::string& err) {
    const int m = P->m, C = P->n_classes;
    float* z = (float*)(ws + P->logits); float* dz = (float*)(ws + P->dlogits); float* rl = (float*)(ws + P->row_loss);
    if (C <= 128) {
        RUN(dsspk_fc_softmax_xent(s, a, w + fw, w + fb, y, z, dz, rl, m, n_in, C));
        RUN(dsspk_fc_bwd(s, a, dz, w + fw, g + fw, g + fb, d_in, mask, rl, loss, m, n_in, C));
    } else {                    // more classes than the fused kernel holds
        RUN(dsspk_gemm(s, a, n_in, 1, w + fw, C, 1, z, C, m, C, n_in, w + fb, 0));
        RUN(dsspk_softmax_xent(s, z, y, dz, loss, m, C));
        RUN(dsspk_fc_bwd(s, a, dz, w + fw, g + fw, g + fb, d_in, mask, nullptr, nullptr, m, n_in, C));
    }
    return 0;
}

int step_mlp(Plan* P, char* ws, void* s, const float* x, const int32_t* y, const float* w, float* g, float* loss, std::string& err) {
    const int m = P->m, C = P->n_classes;
    float* a1 = (float*)(ws + P->mlp_a1); float* da1 = (float*)(ws + P->mlp_da1);
    const int64_t w1 = 0, b1 = 3072 * 256, w2 = b1 + 256, b2 = w2 + 256 * (int64_t)C;
    RUN(dsspk_gemm(s, x, 3072, 1, w + w1, 256, 1, a1, 256, m, 256, 3072, w + b1, 1));
    if (int rc = last_layer(P, ws, s, a1, 256, y, w, g, w2, b2, da1, 1, loss, err)) return rc;
    RUN(dsspk_fc_bwd(s, x, da1, nullptr, g + w1, g + b1, nullptr, 0, nullptr, nullptr, m, 3072, 256));
    return 0;
}

int step_alexnet(Plan* P, char* ws, void* s, const float* x, const int32_t* y, const float* w, float* g, float* loss, std::string& err) {
    const int m = P->m, C = P->n_classes;
    auto F = [&](size_t off) { return (float*)(ws + off); };
    float *a1 = F(P->ax_a1), *p1 = F(P->ax_p1), *a2 = F(P->ax_a2), *p2 = F(P->ax_p2), *a3 = F(P->ax_a3), *a4 = F(P->ax_a4);
    uint8_t *arg1 = (uint8_t*)(ws + P->ax_arg1), *arg2 = (uint8_t*)(ws + P->ax_arg2);
    float *da4 = F(P->ax_da4), *da3 = F(P->ax_da3), *dp2 = F(P->ax_dp2);
    float *da2 = F(P->ax_da2), *dp1 = F(P->ax_dp1), *scr = F(P->wg_scratch);
    const int64_t cw1 = 0, cb1 = 4800, cw2 = cb1 + 64, cb2 = cw2 + 102400, fw1 = cb2 + 64, fb1 = fw1 + 3136 * 384,
                  fw2 = fb1 + 384, fb2 = fw2 + 384 * 192, fw3 = fb2 + 192, fb3 = fw3 + 192 * (int64_t)C;
    // forward
    SplitFilterJob filters;
    filters.add(w + cw2, ws + P->wide2.fwd, ws + P->wide2.bwd, 64, 5);
    RUN(conv_first_pool_fwd((hipStream_t)s, x, w + cw1, w + cb1, a1, p1, arg1, m, filters));
    RUN(dsspk_conv_split_fwd(s, p1, ws + P->wide2.fwd, w + cb2, a2, m, 15, 15, 64, 64, 5, 2, 1));
    RUN(dsspk_maxpool_fwd(s, a2, p2, arg2, m, 15, 15, 64));
    RUN(dsspk_gemm(s, p2, 3136, 1, w + fw1, 384, 1, a3, 384, m, 384, 3136, w + fb1, 1));
    RUN(dsspk_gemm(s, a3, 384, 1, w + fw2, 192, 1, a4, 192, m, 192, 384, w + fb2, 1));
    if (int rc = last_layer(P, ws, s, a4, 192, y, w, g, fw3, fb3, da4, 1, loss, err)) return rc;
    // backward; the convolutions' partial filter gradients wait for one launch at the end
    jobs::Partials waiting[2];
    RUN(dsspk_fc_bwd(s, a3, da4, w + fw2, g + fw2, g + fb2, da3, 1, nullptr, nullptr, m, 384, 192));
    RUN(dsspk_fc_bwd(s, p2, da3, w + fw1, g + fw1, g + fb1, dp2, 0, nullptr, nullptr, m, 3136, 384));
    RUN(dsspk_maxpool_bwd_relu(s, dp2, arg2, a2, da2, m, 15, 15, 64));
    RUN(conv_split_bwd_weight_parts((hipStream_t)s, p1, da2, g + cw2, 1, F(P->wide2.partial), m, 15, 15, 64, 64, 5, 2, &waiting[1]));      // and the biases behind the filter
    RUN(dsspk_conv_split_bwd_data(s, da2, ws + P->wide2.bwd, nullptr, dp1, m, 15, 15, 64, 64, 5, 2));
    RUN(conv_first_pool_bwd_weight_parts((hipStream_t)s, x, dp1, p1, arg1, g + cw1, scr, m, &waiting[0]));      // and the biases behind the filter
    return wgrad_reduce_many((hipStream_t)s, 2, waiting);
}

// The reduced AlexNet with three convolutional and two fully connected layers (Sec. V-A3); the layers and kernels of
// step_alexnet in a different order.
int step_alexnet3(Plan* P, char* ws, void* s, const float* x, const int32_t* y, const float* w, float* g, float* loss, std::string& err) {
    const int m = P->m, C = P->n_classes;
    auto F = [&](size_t off) { return (float*)(ws + off); };
    float *a1 = F(P->ax_a1), *p1 = F(P->ax_p1), *a2 = F(P->ax_a2), *p2 = F(P->ax_p2), *c3 = F(P->ax_c3), *a3 = F(P->ax_a3);
    uint8_t *arg1 = (uint8_t*)(ws + P->ax_arg1), *arg2 = (uint8_t*)(ws + P->ax_arg2);
    float *da3 = F(P->ax_da3), *dc3 = F(P->ax_dc3), *dp2 = F(P->ax_dp2);
    float *da2 = F(P->ax_da2), *dp1 = F(P->ax_dp1), *scr = F(P->wg_scratch);
    const int64_t cw1 = 0, cb1 = 4800, cw2 = cb1 + 64, cb2 = cw2 + 102400, cw3 = cb2 + 64, cb3 = cw3 + 36864,
                  fw1 = cb3 + 64, fb1 = fw1 + 3136 * 384, fw2 = fb1 + 384, fb2 = fw2 + 384 * (int64_t)C;
    // forward
    SplitFilterJob filters;
    filters.add(w + cw2, ws + P->wide2.fwd, ws + P->wide2.bwd, 64, 5);
    filters.add(w + cw3, ws + P->wide3.fwd, ws + P->wide3.bwd, 64, 3);
    RUN(conv_first_pool_fwd((hipStream_t)s, x, w + cw1, w + cb1, a1, p1, arg1, m, filters));
    RUN(dsspk_conv_split_fwd(s, p1, ws + P->wide2.fwd, w + cb2, a2, m, 15, 15, 64, 64, 5, 2, 1));
    RUN(dsspk_maxpool_fwd(s, a2, p2, arg2, m, 15, 15, 64));
    RUN(dsspk_conv_split_fwd(s, p2, ws + P->wide3.fwd, w + cb3, c3, m, 7, 7, 64, 64, 3, 1, 1));
    RUN(dsspk_gemm(s, c3, 3136, 1, w + fw1, 384, 1, a3, 384, m, 384, 3136, w + fb1, 1));
    if (int rc = last_layer(P, ws, s, a3, 384, y, w, g, fw2, fb2, da3, 1, loss, err)) return rc;
    // backward, as above
    jobs::Partials waiting[3];
    RUN(dsspk_fc_bwd(s, c3, da3, w + fw1, g + fw1, g + fb1, dc3, 1, nullptr, nullptr, m, 3136, 384));
    RUN(conv_split_bwd_weight_parts((hipStream_t)s, p2, dc3, g + cw3, 1, F(P->wide3.partial), m, 7, 7, 64, 64, 3, 1, &waiting[2]));
    RUN(dsspk_conv_split_bwd_data(s, dc3, ws + P->wide3.bwd, nullptr, dp2, m, 7, 7, 64, 64, 3, 1));
    RUN(dsspk_maxpool_bwd_relu(s, dp2, arg2, a2, da2, m, 15, 15, 64));
    RUN(conv_split_bwd_weight_parts((hipStream_t)s, p1, da2, g + cw2, 1, F(P->wide2.partial), m, 15, 15, 64, 64, 5, 2, &waiting[1]));      // and the biases behind the filter
    RUN(dsspk_conv_split_bwd_data(s, da2, ws + P->wide2.bwd, nullptr, dp1, m, 15, 15, 64, 64, 5, 2));
    RUN(conv_first_pool_bwd_weight_parts((hipStream_t)s, x, dp1, p1, arg1, g + cw1, scr, m, &waiting[0]));      // and the biases behind the filter
    return wgrad_reduce_many((hipStream_t)s, 3, waiting);
}

constexpr int LARGE_ABOVE = 96;
// A record buffer holds 512 records of 16 channels, four an image.  A convolution of more images would write beyond it, and the one behind would
// refuse so many.
constexpr int RESNET_MAX = 128;

int step_resnet(Plan* P, char* ws, void* s, const float* x, const int32_t* y, const float* w, float* g, float* loss, std::string& err) {
    const int m = P->m;
    if (m > RESNET_MAX) { err = "residual networks take at most 128 images"; return -1; }
    const float eps = 1e-5f;
    auto F = [&](size_t off) { return (float*)(ws + off); };
    float* bscr = F(P->bn_scratch);
    // ---- forward
    // Statistics records ping-pong between two buffers: conv1 writes recA, conv2 reads recA and writes recB,
    // the next block's conv1 reads recB.  A "regular" block (stride 1, same width, shape covered by the specialised
    // kernels) has its two batch norms folded into the loaders of the convolutions that consume them:
    //   conv1 [+ BN2/shortcut/ReLU of the previous block in its loader]  ->  conv2 [+ BN1/ReLU in its loader]
    // and only the last block of a run materialises its output with the stand-alone BN kernels.
    float *recA = bscr, *recB = F(P->bn_scratch2);
    float *g0 = F(P->G[0]), *g1 = F(P->G[1]), *g2 = F(P->G[2]);     // backward; g0: gradient w.r.t. the current block output
    const int nb = (int)P->blocks.size();
    // Above LARGE_ABOVE images the larger workgroups of dsspk_conv3x3_large_*: half as many records, few enough for every workgroup to
    // add up (173 launches of a 110-layer step less).  A round with the four-wavefront / the larger ones, us: 20 layers, one worker, batch 65
    // 660 / 661, four workers 80 1467 / 1416, 96 1571 / 1500; 50 layers, eight workers 65 5108 / 4892, 96 5977 / 5676; 110 layers 80 11673 / 11055;
    // before the filters were converted ahead: 20 layers, four workers 97 1603 / 1532, 128 1804 / 1744, 50 layers, eight workers 97 7550 / 7090,
    // 128 8500 / 8090, 110 layers 128 17280 / 16680.  By these figures the line belongs at 64 (not lower: up to 64 images the first stride-2
    // convolution leaves more records than they add up); it lies at 96 because from 65 to 96 images a step would then take its statistics and filter
    // gradients from other partial sums, which no test checks at those batches yet.
    // Up to DSSPK_CONV3X3_SMALL_MAX images the smaller workgroups of dsspk_conv3x3_small_* (k_conv3x3_small.hip: 5 to 8 % of a step).
    const bool large = m > LARGE_ABOVE && m <= DSSPK_CONV3X3_LARGE_MAX, small = m <= DSSPK_CONV3X3_SMALL_MAX;
    auto parts_of = [&](int H, int cin, int cout, int stride) {       // records that the forward convolution leaves
        if (cin != cout || stride != 1) return dsspk_conv_fwd_records_parts(m, H, H, cin, cout, 3, 3, stride, 1);
        return large   ? dsspk_conv3x3_large_parts(m, H, cin)
               : small ? dsspk_conv3x3_small_parts(m, H, cin)
                       : dsspk_conv_fwd_stat_parts(m, H, H, cin, cout, 3, 3, stride, 1);
    };
    uint4* planes = (uint4*)(ws + P->filters);
    auto forward_filter = [&](int64_t at, size_t f) { return Filter3x3(w + at, planes + f); };
    auto input_filter = [&](int64_t at, size_t f, int C) { return Filter3x3(w + at, planes + f + filter3x3_uint4s(C)); };
    auto conv = [&](const float* src, const Filter3x3& wt, float* dst, int H, int cin, int cout, int stride, float* rec) {
        if (rec && (cin != cout || stride != 1)) return dsspk_conv_fwd_records(s, src, wt.w, dst, rec, m, H, H, cin, cout, 3, 3, stride, 1);
        if ((large || small) && rec)
            return (large ? conv3x3_large_fwd : conv3x3_small_fwd)(s, src, nullptr, 0, nullptr, nullptr, 0.f, nullptr, nullptr, nullptr, wt,
                                                                              dst, rec, 0, m, H, cin);
        if (rec) return conv3x3_tiled((hipStream_t)s, src, wt, nullptr, dst, rec, m, H, cin, false);
        return dsspk_conv_fwd(s, src, wt.w, nullptr, dst, m, H, H, cin, cout, 3, 3, stride, 1, 0, nullptr);
    };
    auto conv_prebn = [&](const float* src, const float* rec, int parts, const float* gamma, const float* beta, const float* shortcut, float* act,
                          float* stats, const Filter3x3& wt, float* dst, float* rec_out, int H, int C, bool half = false) {
        if (large || small)
            return (large ? conv3x3_large_fwd : conv3x3_small_fwd)(s, src, rec, parts, gamma, beta, eps, shortcut, act, stats, wt, dst,
                                                                              rec_out, half, m, H, C);
        return conv3x3_tiled_prebn((hipStream_t)s, src, rec, parts, gamma, beta, eps, shortcut, half, act, stats, wt, dst, rec_out, m, H, C);
    };
    auto regular = [&](int i) {
        const ResBlock& b = P->blocks[i];
        return b.stride == 1 && b.cin == b.cout && parts_of(b.H, b.cin, b.cout, 1) > 0;
    };
    // The stem's batch norm is folded into the first block's convolution in the same way where the stem leaves records.
    // It leaves 16 an image, of which the smaller workgroups add up at most 256; beyond 32 images it leaves some at 64 alone, where its tiles get
    // larger and the list just fits (20 layers, one worker, batch 63 / 64 / 65: 654 / 641 / 687 us; at 65 the first stride-2 convolution's list ends
    // as well).
    const int stem_parts = small && m > 16 ? 0 : parts_of(32, 3, 16, 1);
    RUN(conv_stem((hipStream_t)s, x, w + P->stem_w, F(P->stem_c), stem_parts ? recB : nullptr, m, FilterJob(w, planes, P->filter_runs)));
    if (!stem_parts)
        RUN(dsspk_bn_fwd(s, F(P->stem_c), w + P->stem_g, w + P->stem_b, F(P->stem_a), F(P->stem_st), bscr, (long)m * 1024, 16, eps, 1, 0, nullptr, 0, 0,
                         0, 0));
    // everything between the last convolution and its gradient in one launch
    const bool head = resnet_head_takes(m, parts_of(8, 64, 64, 1), P->n_classes);
    const float* cur = F(P->stem_a);
    bool pending = stem_parts > 0;   // the previous block's output is not written yet (its BN2 is folded into this conv1)
    for (int bi = 0; bi < nb; ++bi) {
        const ResBlock& B = P->blocks[bi];
        const int Ho = B.H / B.stride;
        const long M = (long)m * Ho * Ho;
        const int mode = (B.stride == 1 && B.cin == B.cout) ? 1 : 2;
        const int parts1 = parts_of(B.H, B.cin, B.cout, B.stride);
        const int parts2 = parts_of(Ho, B.cout, B.cout, 1);
        if (pending && bi == 0) {
            RUN(conv_prebn(F(P->stem_c), recB, stem_parts, w + P->stem_g, w + P->stem_b, nullptr, F(P->stem_a), F(P->stem_st), forward_filter(B.w1, B.f1), F(B.c1), recA, 32,
                           16));
        } else if (pending) {
            const ResBlock& Pv = P->blocks[bi - 1];
            const float* pin = bi >= 2 ? F(P->blocks[bi - 2].out) : F(P->stem_a);         // the previous block's input = its shortcut
            RUN(conv_prebn(F(Pv.c2), recB, parts2, w + Pv.g2, w + Pv.b2, pin, F(Pv.out), F(Pv.st2), forward_filter(B.w1, B.f1), F(B.c1), recA, B.H, B.cin, Pv.stride == 2));
        } else {
            RUN(conv(cur, mode == 1 ? forward_filter(B.w1, B.f1) : Filter3x3(w + B.w1), F(B.c1), B.H, B.cin, B.cout, B.stride, parts1 ? recA : nullptr));
        }
        if (parts1 && parts2) {
            RUN(conv_prebn(F(B.c1), recA, parts1, w + B.g1, w + B.b1, nullptr, F(B.a1), F(B.st1), forward_filter(B.w2, B.f2), F(B.c2), recB, Ho, B.cout));
        } else {
            RUN(dsspk_bn_fwd(s, F(B.c1), w + B.g1, w + B.b1, F(B.a1), F(B.st1), recA, M, B.cout, eps, 1, 0, nullptr, 0, 0, 0, parts1));
            RUN(conv(F(B.a1), forward_filter(B.w2, B.f2), F(B.c2), Ho, B.cout, B.cout, 1, parts2 ? recB : nullptr));
        }
        pending = parts2 > 0 && bi + 1 < nb && regular(bi + 1);
        if (bi + 1 == nb && head) {
            const HeadArgs end = {F(B.out), F(B.st2), y, F(P->pooled), F(P->logits), F(P->dlogits), F(P->row_loss), g0, recA,
                                  eps, 1.f / (float)m, (int)(M / parts2), P->n_classes};
            RUN(resnet_head((hipStream_t)s, F(B.c2), recB, parts2, w + B.g2, cur, mode == 2, w + P->fc_w, m, end));
        } else if (bi + 1 == nb) {
            RUN(dsspk_bn_fwd_gap(s, F(B.c2), w + B.g2, w + B.b2, F(B.out), F(B.st2), recB, parts2, cur, mode == 2, F(P->pooled), m, Ho, B.cout, eps));
        } else if (!pending) {
            RUN(dsspk_bn_fwd(s, F(B.c2), w + B.g2, w + B.b2, F(B.out), F(B.st2), recB, M, B.cout, eps, 1, mode, cur, m, Ho, Ho, parts2));
        }
        cur = F(B.out);
    }
    if (head) {
        RUN(dsspk_fc_bwd(s, F(P->pooled), F(P->dlogits), nullptr, g + P->fc_w, g + P->fc_b, nullptr, 0, F(P->row_loss), loss, m, 64, P->n_classes));
    } else if (int rc = last_layer(P, ws, s, F(P->pooled), 64, y, w, g, P->fc_w, P->fc_b, F(P->dpooled), 0, loss, err)) {
        return rc;
    }
    // ---- backward
    // Per convolution layer the backward pass is  BN backward -> d-input convolution -> d-filter convolution.
    // Where the specialised 3x3 kernels apply, and the gradient arrives already masked with sum records (written by the
    // epilogue of the d-input convolution before it), these collapse (regular_layer below):
    //   stages 1-2: ONE kernel - BN backward in its loader, d-input convolution, ReLU mask + sum records of the
    //               next batch norm in its epilogue, and the d-filter partial sums from the same LDS tiles (dx is
    //               never stored) - followed by the small kernel that sums those records
    //   stage 3   : the d-input kernel (stores dx), then the d-filter kernel, which carries the sums job; up to 32 images one kernel too
    // In both forms the d-input kernel carries the reduction of an earlier layer's d-filter partial sums, the oldest that waits.  A layer
    // whose d-filter kernel is of another kind leaves its partial sums waiting too; what waits at the end is one launch.
    // Everything else (stem, first convolutions of the stride-2 blocks) takes the stand-alone kernels.
    //   parts0 > 0 : g0 holds the masked dz of this block's BN2 and recB0 its records
    //   tot0       : their sums are in totB already (and dgamma / dbeta of BN2 stored), or the kernel behind adds them up
    //   pend       : d-filter partial sums whose reduction has not been launched yet, the oldest first
    // (the head reads its input's records from the one record buffer and leaves its own in the other: the two change places)
    float *recB0 = head ? recA : recB, *recA0 = head ? recB : recA, *totA = F(P->tot_a), *totB = F(P->tot_b);
    float* scrs[WG_SCRATCH] = {F(P->wg_scratch)};
    for (int i = 1; i < WG_SCRATCH; ++i) scrs[i] = F(P->wg_more[i - 1]);
    int parts0 = 0;
    bool tot0 = false;
    struct Pending { jobs::Partials p[WG_SCRATCH]; int n; } pend = {};
    auto free_scr = [&]() {
        int i = 0;
        for (int k = 0; k < pend.n; ++k)
            if (pend.p[k].partial == scrs[i]) { ++i; k = -1; }
        return scrs[i];
    };
    auto push_back = [&](const float* partial, float* dw, int E, int chunks, bool quads = false) { pend.p[pend.n++] = {partial, dw, E, chunks, quads}; };
    auto pop_front = [&]() {
        --pend.n;
        for (int k = 0; k < pend.n; ++k) pend.p[k] = pend.p[k + 1];
    };
    auto flush = [&]() -> int {
        const int n = pend.n;
        pend.n = 0;
        return n ? wgrad_reduce_many((hipStream_t)s, n, pend.p) : 0;
    };
    // d-filter of a layer with a kernel of its own; its partial sums wait
    auto filter_grad = [&](const float* xi, const float* dy, float* dw, int H, int cin, int cout, int stride) -> int {
        if (pend.n == WG_SCRATCH - 1) RUN(flush());
        int chunks = 0;
        float* to = free_scr();
        RUN(dsspk_conv_bwd_weight_parts(s, xi, dy, to, m, H, H, cin, cout, 3, 3, stride, 1, nullptr, 0, 0, nullptr, nullptr, nullptr, &chunks));
        push_back(to, dw, 9 * cin * cout, chunks);
        return 0;
    };
    // dz (masked, records summed into tot) -> through BN (xc, st, gamma) -> dx -> d-input (+ add) with the mask / records
    // epilogue (mask_src = x_in, xc_post, st_post -> records) into out, and d-filter (x_in, dx) into dw (pending).
    // The sums of dz: in_rec / in_parts / in_dgamma / in_dbeta, added up by the kernel itself in the larger and the smaller workgroups; between
    // them (33 images and more: more records than a workgroup of those kernels adds up) already in tot (ready) or by a launch here, and
    // gamma_post, beta_post: of the batch norm of xc_post, if x_in is ReLU(BN(xc_post)) with nothing added; sum_next: the records just written are summed into ntot / ndgamma / ndbeta for the next layer.
    auto regular_layer = [&](const float* in_rec, int in_parts, float* in_dgamma, float* in_dbeta, bool ready,
                             const float* dz, const float* xc, const float* st, const float* gamma, float* tot,
                             const Filter3x3& wt, const float* add, float* out, const float* x_in, const float* xc_post,
                             const float* st_post, float* records, float* dw, int H, int Cc, bool sum_next, int nparts,
                             float* ntot, float* ndgamma, float* ndbeta, const float* gamma_post = nullptr, const float* beta_post = nullptr) -> int {
        float* out_scr = free_scr();
        const jobs::Partials red = pend.n ? pend.p[0] : jobs::Partials{};
        if (pend.n) pop_front();
        if (large || small) {
            int chunks = parts_of(H, Cc, Cc, 1);
            const auto bwd = large ? conv3x3_large_bwd : conv3x3_small_bwd;
            const bool apart = large && Cc == 64;           // a d-filter kernel of its own
            RUN(bwd(s, dz, xc, st, gamma, in_rec, in_parts, in_dgamma, in_dbeta, apart ? g1 : nullptr, apart ? nullptr : out_scr, wt, add, out,
                    x_in, xc_post, st_post, records, red, m, H, Cc, gamma_post, beta_post));
            if (apart) RUN(dsspk_conv_bwd_weight_parts(s, x_in, g1, out_scr, m, H, H, Cc, Cc, 3, 3, 1, 1, nullptr, 0, 0, nullptr, nullptr, nullptr, &chunks));
            push_back(out_scr, dw, 9 * Cc * Cc, chunks, small && Cc == 64);
            return 0;
        }
        if (!ready) RUN(dsspk_bn_bwd_totals(s, in_rec, in_parts, Cc, tot, in_dgamma, in_dbeta));
        int chunks = dsspk_conv_bwd_fused_chunks(m, H, Cc);
        if (chunks > 0) {
            RUN(conv3x3_tiled_dgrad_bn_wgrad((hipStream_t)s, dz, xc, st, gamma, tot, in_rec, in_parts, in_dgamma, in_dbeta, wt, add, out, xc_post,
                                             st_post, records, x_in, out_scr, red.partial, red.dw, red.E, red.chunks, m, H, Cc, gamma_post, beta_post));
            if (sum_next) RUN(dsspk_bn_bwd_totals(s, records, nparts, Cc, ntot, ndgamma, ndbeta));
        } else {
            RUN(conv3x3_tiled_dgrad_bn((hipStream_t)s, dz, xc, st, gamma, tot, in_rec, in_parts, in_dgamma, in_dbeta, g1, wt, add, out, x_in,
                                       xc_post, st_post, records, red.partial, red.dw, red.E, red.chunks, m, H, Cc, gamma_post, beta_post));
            RUN(dsspk_conv_bwd_weight_parts(s, x_in, g1, out_scr, m, H, H, Cc, Cc, 3, 3, 1, 1, sum_next ? records : nullptr,
                                            nparts, Cc, ntot, ndgamma, ndbeta, &chunks));
        }
        push_back(out_scr, dw, 9 * Cc * Cc, chunks);
        return 0;
    };
    for (int bi = (int)P->blocks.size() - 1; bi >= 0; --bi) {
        const ResBlock& B = P->blocks[bi];
        const float* xin = bi ? F(P->blocks[bi - 1].out) : F(P->stem_a);
        const int Ho = B.H / B.stride;
        const long M = (long)m * Ho * Ho;
        const int parts1 = parts_of(Ho, B.cout, B.cout, 1);
        const bool identity = B.stride == 1 && B.cin == B.cout;
        const int partsp = identity ? parts_of(B.H, B.cin, B.cout, 1) : 0;
        const bool fused1 = parts1 > 0 && partsp > 0;        // conv1's layer takes the two-launch form
        // ---- BN2 + conv2: g0 = dz2 -> g1 = d conv2 output, g2 = dz1 = d a1 * [a1 > 0] (+ BN1's records in recA0)
        if (bi + 1 == nb && head) {
            parts0 = m;
        } else if (bi + 1 == nb) {      // from the pooled gradient
            RUN(dsspk_gap_bwd_bn_reduce(s, F(P->dpooled), F(B.c2), F(B.st2), F(B.out), g0, recB0, m, Ho, B.cout));
            parts0 = m;
        } else if (!parts0) {           // g0 is not masked yet
            RUN(dsspk_bn_bwd_reduce_parts(s, F(B.c2), F(B.st2), g0, F(B.out), recB0, parts1, M, B.cout));
            parts0 = parts1;
            tot0 = false;
        }
        RUN(regular_layer(recB0, parts0, g + B.g2, g + B.b2, tot0, g0, F(B.c2), F(B.st2), w + B.g2, totB, input_filter(B.w2, B.f2, B.cout), nullptr, g2, F(B.a1), F(B.c1), F(B.st1), recA0,
                          g + B.w2, Ho, B.cout, fused1, parts1, totA, g + B.g1, g + B.b1, w + B.g1, w + B.b1));        // sums of BN1's records to totA if fused1
        // ---- BN1 + conv1: g2 = dz1 -> g1 = d conv1 output; d-input (+ dz2 through an identity shortcut) = gradient
        //      w.r.t. the block's input, which is the previous block's (or the stem's) post-ReLU output: mask +
        //      records of ITS batch norm in the same kernel where the specialised kernel applies
        if (fused1) {
            const float* pc = bi ? F(P->blocks[bi - 1].c2) : F(P->stem_c);
            const float* pst = bi ? F(P->blocks[bi - 1].st2) : F(P->stem_st);
            // output in place over the shortcut's gradient g0; g0 stays the gradient w.r.t. the previous block's output
            const bool next_fused = bi > 0;                  // the previous block's conv2 has this convolution's shape
            RUN(regular_layer(recA0, parts1, g + B.g1, g + B.b1, true, g2, F(B.c1), F(B.st1), w + B.g1, totA, input_filter(B.w1, B.f1, B.cout), g0, g0, xin, pc, pst, recB0, g + B.w1, B.H, B.cin,
                              next_fused, partsp, totB, next_fused ? g + P->blocks[bi - 1].g2 : nullptr,
                              next_fused ? g + P->blocks[bi - 1].b2 : nullptr));
            parts0 = partsp;
            tot0 = next_fused;
        } else {                        // first block of a stage: stride 2, shortcut without parameters
            RUN(dsspk_bn_bwd_dx(s, F(B.c1), w + B.g1, F(B.st1), g2, g1, g + B.g1, g + B.b1, recA0, M, B.cout, parts1));
            // both gradients, with the ReLU and the sums of the block in front, in one kernel where the kernel behind adds up as many records itself
            parts0 = small ? conv_stride2_bwd_records(m, B.H, B.cin) : 0;
            if (parts0 > conv3x3_small_records(B.cin)) parts0 = 0;
            if (parts0) {
                const ResBlock& Pv = P->blocks[bi - 1];
                if (pend.n == WG_SCRATCH - 1) RUN(flush());
                float* to = free_scr();
                int chunks = 0;
                RUN(conv_stride2_bwd((hipStream_t)s, g1, w + B.w1, g0, g2, to, BehindBn{xin, F(Pv.c2), F(Pv.st2), recB0}, m, B.H, B.cin, &chunks));
                push_back(to, g + B.w1, 9 * B.cin * B.cout, chunks);
            } else {
                RUN(filter_grad(xin, g1, g + B.w1, B.H, B.cin, B.cout, B.stride));
                RUN(dsspk_conv_bwd_data_shortcut(s, g1, w + B.w1, g0, g2, m, B.H, B.H, B.cin, B.cout, 3, 3, 1));
            }
            tot0 = false;
            float* t = g0; g0 = g2; g2 = t;
        }
    }
    RUN(dsspk_bn_bwd_dx(s, F(P->stem_c), w + P->stem_g, F(P->stem_st), g0, g1, g + P->stem_g, g + P->stem_b, recB0,
                        (long)m * 1024, 16, parts0));
    RUN(filter_grad(x, g1, g + P->stem_w, 32, 3, 16, 1));
    return flush();
}

}  // namespace

Plan* create(int model_id, int batch, int n_classes, int K, void* workspace_dev, std::string& err) {
    Plan* P = new Plan();
    if (!P->build(model_id, batch, n_classes)) { err = "unknown model"; delete P; return nullptr; }
    if (batch > 1024 || n_classes > 1024) { err = "batch and n_classes must be <= 1024"; delete P; return nullptr; }
    P->K = K;
    P->ws = (char*)workspace_dev;
    return P;
}

void destroy(Plan* p) { delete p; }

int step(Plan* P, int worker, hipStream_t stream, const float* x, const int32_t* y, const float* w, float* g, float* loss,
         std::string& err) {
    char* ws = P->ws + (size_t)worker * P->per_worker;
    if (P->model_id == DSSP_MODEL_MLP) return step_mlp(P, ws, stream, x, y, w, g, loss, err);
    if (P->model_id == DSSP_MODEL_ALEXNET_DS) return step_alexnet(P, ws, stream, x, y, w, g, loss, err);
    if (P->model_id == DSSP_MODEL_ALEXNET_3C) return step_alexnet3(P, ws, stream, x, y, w, g, loss, err);
    return step_resnet(P, ws, stream, x, y, w, g, loss, err);
}

}  // namespace dssp_model

extern "C" int64_t dssp_model_param_count(int model_id, int n_classes) {
    dssp_model::Plan P;
    if (n_classes < 2 || !P.build(model_id, 1, n_classes)) return -1;
    return P.n_params;
}

extern "C" int dssp_model_segments(int model_id, int n_classes, int32_t* kind, int64_t* size, int64_t* fan_in, int max_segments) {
    dssp_model::Plan P;
    if (n_classes < 2 || !P.build(model_id, 1, n_classes)) return DSSP_EINVAL;
    const int n = (int)P.segs.size();
    for (int i = 0; i < n && i < max_segments; ++i) {
        if (kind) kind[i] = P.segs[i].kind;
        if (size) size[i] = P.segs[i].size;
        if (fan_in) fan_in[i] = P.segs[i].fan_in;
    }
    return n;
}

extern "C" size_t dssp_workspace_bytes(int model_id, int batch, int n_classes, int K) {
    dssp_model::Plan P;
    if (model_id == DSSP_MODEL_NONE) return 0;
    if (n_classes < 2 || batch < 1 || K < 1 || !P.build(model_id, batch, n_classes)) return 0;
    return P.per_worker * (size_t)K;
}

extern "C" int dssp_workspace_tensor(int model_id, int batch, int n_classes, int K, int worker, int what, int index,
                                     size_t* byte_offset, int64_t* count) {
    dssp_model::Plan P;
    if (n_classes < 2 || batch < 1 || worker < 0 || worker >= K || !P.build(model_id, batch, n_classes)) return DSSP_EINVAL;
    int seen = 0;
    for (const auto& t : P.tens)
        if (t.what == what) {
            if (seen == index) {
                if (byte_offset) *byte_offset = (size_t)worker * P.per_worker + t.off;
                if (count) *count = t.count;
                return DSSP_OK;
            }
            ++seen;
        }
    return DSSP_EINVAL;
}
