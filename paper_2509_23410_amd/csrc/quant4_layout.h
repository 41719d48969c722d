// Sizes and places inside the 4-bit storage (its byte layout: quant4.hip), and the launch of the prefill kernel with two K groups.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout.h"

namespace patch {

__host__ __device__ constexpr int q4_dense_codes(int t) { return t * t / 2; }
__host__ __device__ constexpr int q4_sparse_codes(int t) { return t * t / 4; }
__host__ __device__ constexpr int q4_sparse_pos(int t) { return t * t / 8; }
__host__ __device__ constexpr int q4_round_up(int b) { return (b + kGranule - 1) / kGranule * kGranule; }
__host__ __device__ constexpr int q4_dense_tile(int t) { return q4_round_up(q4_dense_codes(t)); }
__host__ __device__ constexpr int q4_sparse_tile(int t) { return q4_round_up(q4_sparse_codes(t) + q4_sparse_pos(t)); }
// scale of row r (0..15) of strip `strip` (over the whole matrix) for tile column tk
__host__ __device__ constexpr int64_t q4_scale_index(int64_t strip, int Tk, int tk, int r) { return (strip * Tk + tk) * 16 + r; }

constexpr int64_t kKgMaxK = 1 << 24;   // prefill4_kgroups_kernel: lane offsets into the 128 rows of X have 32 bits
struct Q4Prefill {
    const uint16_t* X;
    int64_t M, N, K;
    int tile, Tk;
    const uint8_t* payload;
    const uint16_t* scales;
    const uint32_t* table;
    float* Y;
};
constexpr size_t kKgSlotBytes = 128 * 256 * sizeof(float);
// tail = 0: the whole product in `split` K slices, more than one to ws (split x M x N floats, to be summed).  tail > 0: all blocks of 256 features x 128 rows but the
// last `tail` whole, those in `split` (at least two) slices over slots of kKgSlotBytes each at ws, and their sum.
void launch_prefill4_kgroups(const Q4Prefill& a, int split, int tail, float* ws, hipStream_t stream);

}  // namespace patch
