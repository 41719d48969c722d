// The order in which a prefill launch runs its output tiles.
#pragma once
#include <hip/hip_runtime.h>

namespace patch {

// Tile t of the launch order -> feature block bn (256 features), row block bm (256 rows, or 128 in the kernels of such blocks): groups of 4 row
// blocks x all feature blocks, so that the workgroups an XCD runs at a time cover about 8 feature blocks x 4 row blocks and share both
// operands in its L2.
__device__ __forceinline__ void tile_of(int t, int tiles_n, int tiles_m, int& bn, int& bm) {
    constexpr int GM = 4;
    const int full = (tiles_m / GM) * GM * tiles_n;
    if (t < full) {
        const int g = t / (GM * tiles_n), rem = t % (GM * tiles_n);
        bn = rem / GM;
        bm = g * GM + rem % GM;
    } else {
        const int gm = tiles_m % GM, rem = t - full;
        bn = rem / gm;
        bm = (tiles_m / GM) * GM + rem % gm;
    }
}

}  // namespace patch
