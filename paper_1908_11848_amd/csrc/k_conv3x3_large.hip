// The 3x3 kernels of conv3x3.hpp with eight wavefronts to a workgroup: 16 rows of a 32x32 image with 16 channels, a whole 16x16 image
// with 32, a whole 8x8 image with all 64 output channels.  Against four wavefronts: no (or half the) halo rows, the last stage's input
// loaded and split once and not per half of the output channels, half the partial filter gradients, half the records.
#include "conv3x3_forms.hpp"
#include "../../include/dssp_kernels.h"

namespace {
struct Large { static constexpr int WAVES = 8, TILES = 4, R16 = 16, R32 = 16, SPLIT64 = 1, IMAGES = DSSPK_CONV3X3_LARGE_MAX; };
}  // namespace

DSSPK_CONV3X3_FORM(large, Large)
