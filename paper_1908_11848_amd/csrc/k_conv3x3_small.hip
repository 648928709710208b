// The 3x3 kernels of conv3x3.hpp with four wavefronts of two pixel tiles each: 4 rows of a 32x32 image with 16 channels, 4 rows of a
// 16x16 image with 32, a quarter of the output channels of an 8x8 image with 64.  For batches whose launches leave most compute units idle: a
// launch lasts as long as one workgroup, and these have half the loads, products and stores of the kernels of k_conv3x3.hip.
// Bound by latency: of 6.5 to 13 us a launch 4.5 are what a launch of a graph costs at least.  A push of the 20-layer network, one worker, with
// the kernels of k_conv3x3.hip / these, us: batch 1 488 / 454, 8 512 / 484, 16 543 / 499; four workers, a round: 901 / 853, 954 / 912,
// 1005 / 939; batch 20, 32, one worker 531 / 497, 548 / 518, four 996 / 935, 1047 / 1022; 110 layers, batch 32, eight workers 9275 / 8709.  At
// most 32 images: eight records an image (16 channels) are then all that a workgroup adds up.
#include "conv3x3_forms.hpp"
#include "../../include/dssp_kernels.h"

namespace {
struct Small { static constexpr int WAVES = 4, TILES = 2, R16 = 4, R32 = 4, SPLIT64 = 4, IMAGES = DSSPK_CONV3X3_SMALL_MAX; };
}  // namespace

DSSPK_CONV3X3_FORM(small, Small)

int conv3x3_small_records(int C) { return form_records<Small>(C); }
