// End of a residual network's step (k_head.hip): 64 channels, 8x8 pixels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

constexpr int HEAD_MAX_PARTS = 128, HEAD_MAX_CLASSES = 128;

struct HeadArgs {
    float *out, *stats;                        // the last block's output, and mean, invstd of its second batch norm
    const int32_t* label;
    float *pooled, *logits, *dlogits, *row_loss;
    float *dz, *records_out;                   // masked gradient in front of the last ReLU, its sum records [N][64][2]
    float eps, inv_n;
    int rows_per_record, classes;
};

// Records of the input that every workgroup merges, classes a workgroup holds.
inline bool resnet_head_takes(int N, int parts, int classes) {
    return parts >= 1 && parts <= HEAD_MAX_PARTS && (long)N * 64 % parts == 0 && classes >= 1 && classes <= HEAD_MAX_CLASSES;
}

// x: input of the last batch norm, records: its statistics records; gamma: that norm's gamma and beta, one behind the other; w: [64][classes] and the
// biases behind it.  out, dz and records_out are none of the inputs.
int resnet_head(hipStream_t s, const float* x, const float* records, int parts, const float* gamma, const float* shortcut, bool half, const float* w, int N,
                const HeadArgs& a);
