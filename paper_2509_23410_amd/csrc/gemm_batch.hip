// Hybrid GEMM for batched decoding: up to 128 rows of X per launch (the product Y = X * W_hat^T of Section 4 / Appendix A
// of the paper between its decoding input, a few rows, and its prefill input, thousands).
//
// What bounds it: a compute unit draws about 50 GB/s through its vector L1 here, however many wavefronts ask (one group of
// four or two alike), so a launch needs every compute unit, and what it draws beside the weights counts.  The strip kernel
// (gemm_decode.hip) draws all of X once per 16 features, mid_kernel (gemm_mid.hip) once per 64; here a workgroup owns 128
// features - the weights of a 128-column unit are 20 - 32 KB, its 64 rows of X 16 KB - and X goes through LDS, read there by the
// four wavefronts (two strips each) that multiply the unit.  Two such wavefront groups take the units in turn and add
// their sums in LDS.  Where the groups of 128 features leave compute units idle, gridDim.y workgroups share a group's
// columns and wr_reduce_set_kernel adds their partial sums in order; that second launch costs about 3 us, which is why
// decode_plan (api.hip) weighs it.  f = 0.5, 48 rows, mid_kernel -> this kernel: gate and up of 4096 / 11008 (172 workgroups, no split) 45.4 -> 29.4 us
// (4.8 TB/s of weights), of 5120 / 13824 58.5 -> 40.4; 4096 x 11008 (7 chunks) 22.6 -> 19.9; 5120 x 13824 at 16 rows (strip kernel 36.9; 5 chunks) 22.6.
//
// Beyond 64 rows, up to 128, one wavefront group per workgroup (80 - 128 accumulators and operands of up to eight row blocks per
// lane: 272 - 384 registers): X then costs as much as the weights, still once per 128 features.
//
// Weights go straight into registers in the stored order, one unit ahead, always eight 16-byte loads per wavefront and unit:
// of a 2:4 tile the second load of a step starts at the lane's position word (its first register; the rest is ignored; the
// last lanes read up to 12 bytes into the next tile or the slack behind the payload).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "batch_parts.h"

namespace patch {

// Weights of a unit: [strip][step][operand]; 2:4: operand 0 = values, operand 1 = position word in its first register.
struct BtBf16 {
    template <int TILE>
    struct Unit {
        bt_u32x4 a[2][2][2];
        __device__ __forceinline__ void load(bt_bytes_ptr payload, bt_halves_ptr, int, uint32_t e0, uint32_t e1, int, int, int s0, int lane) {
            const uint32_t v16 = lane * 16, vpos = TILE == 128 ? lane * 4 : (lane >> 1) * 4;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t e = j == 0 ? e0 : e1;
                const bool sp = entry_sparse(e);
                const bt_bytes_ptr base = payload + entry_offset(e);
                const uint32_t vp = sp ? vpos : v16;
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int f = TILE == 128 ? (s0 + s) * 2 + j : s0 + s;   // fragment
                    const int o0 = f * (sp ? kSparseFragBytes : kDenseFragBytes);
                    const int o1 = sp ? sparse_vals_bytes(TILE) + (s0 + s) * (TILE == 128 ? 256 : 128) : o0 + 1024;
                    a[s][j][0] = __builtin_nontemporal_load(reinterpret_cast<const PATCH_BT_GLOBAL bt_u32x4*>(base + o0 + v16));
                    a[s][j][1] = __builtin_nontemporal_load(reinterpret_cast<const PATCH_BT_GLOBAL bt_u32x4*>(base + o1 + vp));
                }
            }
        }
        __device__ __forceinline__ bt_u32x4 operand(int s, int j, int h) const { return a[s][j][h]; }
        // tile 128: a dword holds both steps; tile 64: the dword of the lane and its neighbour
        __device__ __forceinline__ uint32_t positions(int s, int j, int lane) const {
            return TILE == 128 ? (j == 0 ? a[s][0][1][0] : a[s][0][1][0] >> 16) : a[s][j][1][0] >> ((lane & 1) * 16);
        }
    };
};

template <int TILE, int RB, bool SPLIT>
__global__ __launch_bounds__(256 * bt_groups(RB)) void batch_kernel(const uint16_t* __restrict__ X, int64_t m0, int rows, int64_t K, int Tk, const WeightSet set, int ybf16) {
    uint64_t payload64 = reinterpret_cast<uint64_t>(set.payload[0]), table64 = reinterpret_cast<uint64_t>(set.table[0]), Y64 = reinterpret_cast<uint64_t>(set.Y[0]);
    int64_t N = set.N[0];
    int first = 0;
    if (set.count > 1)
#pragma unroll
        for (int i = 1; i < kMaxMany; ++i) {
            const bool here = i < set.count && (int)blockIdx.x >= set.first[i];
            payload64 = here ? reinterpret_cast<uint64_t>(set.payload[i]) : payload64;
            table64 = here ? reinterpret_cast<uint64_t>(set.table[i]) : table64;
            Y64 = here ? reinterpret_cast<uint64_t>(set.Y[i]) : Y64;
            N = here ? set.N[i] : N;
            first = here ? set.first[i] : first;
        }
    const bt_bytes_ptr payload = reinterpret_cast<bt_bytes_ptr>(bt_uniform64(payload64));
    const bt_table_ptr table = reinterpret_cast<bt_table_ptr>(bt_uniform64(table64));
    float* Y = reinterpret_cast<float*>(bt_uniform64(Y64));
    N = (int64_t)bt_uniform64((uint64_t)N);
    const int grp = (int)blockIdx.x - __builtin_amdgcn_readfirstlane(first);
    batch_body<BtBf16, TILE, RB, SPLIT>(X, m0, rows, K, Tk, payload, table, nullptr, Y, N, grp, ybf16);
}

template <int TILE, bool SPLIT>
static void launch_batch_t(const GemmArgs& a, const WeightSet& set, int64_t m0, int rows, int split, int ybf16, hipStream_t stream) {
    const dim3 grid((unsigned)set.units, (unsigned)split);
#define PATCH_BT_CASE(rb)                                                                                                             \
    if (rows <= 16 * rb) {                                                                                                            \
        hipLaunchKernelGGL((batch_kernel<TILE, rb, SPLIT>), grid, dim3(256 * bt_groups(rb)), 0, stream, a.X, m0, rows, a.K, a.Tk, set, ybf16); \
        return;                                                                                                                       \
    }
    PATCH_BT_CASE(1) PATCH_BT_CASE(2) PATCH_BT_CASE(3) PATCH_BT_CASE(4) PATCH_BT_CASE(5) PATCH_BT_CASE(6) PATCH_BT_CASE(8)
#undef PATCH_BT_CASE
}

// Up to kBatchRows rows of X starting at row m0.  set.units / first[] count groups of 128 features, each weight rounded up.  A K split
// (split > 1, at most ceil(K / 128)) needs a.ws with room for split x rows x N floats of every weight.
void launch_batch_set(const GemmArgs& a, const WeightSet& set, int64_t m0, int rows, int split, hipStream_t stream) {
    if (split < 2) {
        if (a.tile == 128) launch_batch_t<128, false>(a, set, m0, rows, 1, a.ybf16, stream);
        else launch_batch_t<64, false>(a, set, m0, rows, 1, a.ybf16, stream);
        return;
    }
    WeightSet part = set;
    WrReduceSet red = {};
    size_t off = 0;
    for (int i = 0; i < set.count; ++i) {
        part.Y[i] = a.ws + off;
        red.ws[i] = a.ws + off;
        red.Y[i] = a.ybf16 ? reinterpret_cast<float*>(reinterpret_cast<uint16_t*>(set.Y[i]) + m0 * set.N[i]) : set.Y[i] + m0 * set.N[i];
        red.n4[i] = (size_t)rows * (size_t)set.N[i] / 4;
        off += (size_t)split * (size_t)rows * (size_t)set.N[i];
    }
    if (a.tile == 128) launch_batch_t<128, true>(a, part, m0, rows, split, 0, stream);
    else launch_batch_t<64, true>(a, part, m0, rows, split, 0, stream);
    if (set.count == 1) wr_reduce(red.ws[0], red.n4[0], split, red.Y[0], a.ybf16, stream);
    else wr_reduce_set(red, set.count, split, a.ybf16, stream);
}

}  // namespace patch
