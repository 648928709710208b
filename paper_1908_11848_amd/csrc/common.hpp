// Shared by the kernel files: launch checks and small device helpers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define DSSPK_LAUNCH_RC() ((int)hipGetLastError())

typedef float floatx4 __attribute__((ext_vector_type(4)));

static inline int ceil_div(long a, long b) { return (int)((a + b - 1) / b); }

// Number of workgroups that keeps every CU of the chip busy a few times over for a
// bandwidth-bound grid-stride kernel (256 CUs in 8 XCDs; workgroups are dealt to XCDs
// round-robin, so a multiple of 8 keeps the XCDs evenly loaded).
static inline int stream_grid(long items_per_block_total, int cap = 256 * 8) {
    long g = items_per_block_total;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

// Workgroups are handed to the 8 XCDs round-robin (workgroup b runs on XCD b mod 8) and every XCD has an L2 of its
// own.  Tiles that are neighbours in memory share data - halo rows between the bands of an image, the whole input
// tile between the channel splits of a band, dy between the input-channel slices of the last stage's d-filter
// kernel - so consecutive tiles go to ONE XCD: workgroup b takes tile (b mod 8) * (n / 8) + b / 8, and what the
// first of them fetched is in that L2 for the next (without this, halo rows and shared tiles come over the fabric
// once per XCD that touches them: 1.1x to 1.7x the operands' bytes).  Where n is no multiple of 8, the first n mod 8 XCDs take a tile more.
__device__ __forceinline__ int xcd_tile(int block, int n_blocks) {
    constexpr int XCDS = 8;
    const int xcd = block % XCDS;
    return xcd * (n_blocks / XCDS) + min(xcd, n_blocks % XCDS) + block / XCDS;
}
