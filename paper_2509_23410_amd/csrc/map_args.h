// Device side of TileMapArgs, and the report of the packing kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"
#include "layout.h"

namespace patch {

// Table entry of tile `local` of the part, tile `t` of the whole map (both the same in all lanes: scalar loads)
__device__ __forceinline__ uint32_t map_entry(const TileMapArgs& map, int local, int t, size_t dense_bytes, size_t sparse_bytes) {
    const int g = local >> 6, i = local & 63;
    const uint64_t bits = ((uint64_t)map.g[g].dense[1] << 32) | map.g[g].dense[0];
    const uint32_t dense = map.g[g].before + (uint32_t)__builtin_popcountll(bits & ((1ull << i) - 1));
    return make_entry((uint64_t)dense * dense_bytes + (uint64_t)((uint32_t)t - dense) * sparse_bytes, !((bits >> i) & 1));
}

// (every writer writes the same word)
__device__ __forceinline__ void report_not_24(uint32_t* not_24) { __hip_atomic_store(not_24, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }

}  // namespace patch
