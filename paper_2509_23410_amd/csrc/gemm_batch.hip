// Hybrid GEMM for batched decoding: up to 64 rows of X per launch (the product Y = X * W_hat^T of Section 4 / Appendix A
// of the paper between its decoding input, a few rows, and its prefill input, thousands).
//
// What bounds it: a compute unit draws about 50 GB/s through its vector L1 here, however many wavefronts ask (one group of
// four or two alike), so a launch needs every compute unit, and what it draws beside the weights counts.  The strip kernel
// (gemm_decode.hip) draws all of X once per 16 features, mid_kernel (gemm_mid.hip) once per 64; here a workgroup owns 128
// features - the weights of a 128-column unit are 20 - 32 KB, its 64 rows of X 16 KB - and X goes through LDS, read there by the
// four wavefronts (two strips each) that multiply the unit.  Two such wavefront groups take the units in turn and add
// their sums in LDS.  Where the groups of 128 features leave compute units idle, gridDim.y workgroups share a group's
// columns and wr_reduce_set_kernel adds their partial sums in order; that second launch costs about 4 us, which is why
// decode_plan (api.hip) weighs it.  f = 0.5, 47 rows, before -> now: gate and up of 4096 / 11008 (172 workgroups, no split) 46.7 -> 31.4 us
// (4.5 TB/s of weights), of 5120 / 13824 59.0 -> 41.4; 4096 x 11008 (8 chunks) 23.9 -> 21.8; 5120 x 13824 at 16 rows (6 chunks) 37.3 -> 23.5.
//
// Weights go straight into registers in the stored order, one unit ahead, always eight 16-byte loads per wavefront and unit:
// of a 2:4 tile the second load of a step starts at the lane's position word (its first register; the rest is ignored; the
// last lanes read up to 12 bytes into the next tile or the slack behind the payload).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "epilogue.h"
#include "kernels.h"
#include "layout.h"

namespace patch {

typedef __bf16 bt_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bt_bf16x16 __attribute__((ext_vector_type(16)));
typedef float bt_f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int bt_u32x4 __attribute__((ext_vector_type(4)));
union BtA { bt_u32x4 raw; bt_bf16x8 v; };
union BtB { bt_u32x4 raw[2]; bt_bf16x8 h[2]; bt_bf16x16 v; };

#define PATCH_BT_GLOBAL __attribute__((address_space(1)))
#define PATCH_BT_CONST __attribute__((address_space(4)))
typedef const PATCH_BT_CONST uint32_t* bt_table_ptr;
typedef const PATCH_BT_GLOBAL uint8_t* bt_bytes_ptr;

constexpr int kBtFeatures = 128;   // per workgroup: 4 wavefronts x 2 strips
constexpr int kBtUnit = 128;       // columns per unit
constexpr int kBtGroups = 2;       // wavefront groups: each takes every second unit

__device__ __forceinline__ uint64_t bt_uniform64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// weights of a unit: [strip][step][operand]; 2:4: operand 0 = values, operand 1 = position word in its first register
struct BtW { bt_u32x4 a[2][2][2]; };

// RB = 16-row blocks of X.  SPLIT: gridDim.y K-chunks, partial sums to a workspace (set.Y; chunk c at c x rows x N).
template <int TILE, int RB, bool SPLIT>
__global__ __launch_bounds__(256 * kBtGroups) void batch_kernel(const uint16_t* __restrict__ X, int64_t m0, int rows, int64_t K, int Tk, const WeightSet set, int ybf16) {
    constexpr int KG = kBtGroups;
    constexpr int kStage = 2 * RB * 16 * 128;   // two steps x rows x 128 bytes
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[KG * 2 * kStage];
    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), kg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    uint8_t* const lds = lds_all + kg * 2 * kStage;
    const int col = lane & 15, q = lane >> 4;
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
    int64_t n0 = (int64_t)grp * kBtFeatures + 32 * w;     // first feature of the wavefront
    const bool live = n0 < N;
    if (!live) n0 -= 64;                                  // tile 64: the other tile row of the group
    const bt_table_ptr trow = table + (n0 / TILE) * Tk;
    const int s0 = (int)(n0 % TILE) / 16;                 // first strip inside the tile

    const int U = (int)((K + kBtUnit - 1) / kBtUnit);
    const int u0 = SPLIT ? (int)((int64_t)blockIdx.y * U / gridDim.y) : 0;
    const int u1 = SPLIT ? (int)((int64_t)(blockIdx.y + 1) * U / gridDim.y) : U;

    // X: thread -> row tid / 16 of every block of 16, 16-byte chunk tid % 16 of the unit's 256 bytes
    const int xr = tid >> 4, xc = tid & 15;
    const PATCH_BT_GLOBAL uint8_t* xsrc[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        int r = 16 * rb + xr;
        if (r >= rows) r = rows - 1;
        xsrc[rb] = reinterpret_cast<const PATCH_BT_GLOBAL uint8_t*>(reinterpret_cast<uintptr_t>(X)) + ((m0 + r) * K + 8 * xc) * 2;
    }
    const int xdst = (xc >> 3) * (RB * 16 * 128) + xr * 128 + (((xc & 7) ^ ((xr >> 1) & 7)) << 4);
    const int swz = (col >> 1) & 7;
    const int rd0 = col * 128 + ((q ^ swz) << 4), rd1 = col * 128 + (((4 + q) ^ swz) << 4);

    bt_f32x4 acc[2][RB];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[s][rb] = bt_f32x4{0.f, 0.f, 0.f, 0.f};

    const uint32_t v16 = lane * 16, vpos = TILE == 128 ? lane * 4 : (lane >> 1) * 4;
    const int shift = (lane & 1) * 16;
    auto entry = [&](int u, int j) -> uint32_t {   // of step j of unit u (past the end: the last tile)
        int t = TILE == 128 ? u : 2 * u + j;
        t = t < Tk ? t : Tk - 1;
        return trow[t];
    };
    auto load_w = [&](BtW& b, uint32_t e0, uint32_t e1) {
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
                b.a[s][j][0] = __builtin_nontemporal_load(reinterpret_cast<const PATCH_BT_GLOBAL bt_u32x4*>(base + o0 + v16));
                b.a[s][j][1] = __builtin_nontemporal_load(reinterpret_cast<const PATCH_BT_GLOBAL bt_u32x4*>(base + o1 + vp));
            }
        }
    };
    bt_u32x4 xreg[RB];
    auto load_x = [&](int u) {
        const int64_t c = (int64_t)u * (kBtUnit * 2);
        const bool half = (u + 1) * (int64_t)kBtUnit > K;   // (tile 64) only the first step exists
        const int64_t off = c - ((half && xc >= 8) ? 128 : 0);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) xreg[rb] = *reinterpret_cast<const PATCH_BT_GLOBAL bt_u32x4*>(xsrc[rb] + off);
    };
    auto store_x = [&](int stage) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) *reinterpret_cast<bt_u32x4*>(lds + stage * kStage + rb * 2048 + xdst) = xreg[rb];
    };
    auto compute = [&](const BtW& b, uint32_t e0, uint32_t e1, int stage, int steps) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (TILE == 64 && j == 1 && steps < 2) break;
            const uint8_t* xs = lds + stage * kStage + j * (RB * 16 * 128);
            BtB x[RB];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                x[rb].raw[0] = *reinterpret_cast<const bt_u32x4*>(xs + rb * 2048 + rd0);
                x[rb].raw[1] = *reinterpret_cast<const bt_u32x4*>(xs + rb * 2048 + rd1);
            }
            if (entry_sparse(j == 0 ? e0 : e1)) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    BtA a;
                    a.raw = b.a[s][j][0];
                    const uint32_t pos = TILE == 128 ? (j == 0 ? b.a[s][0][1][0] : b.a[s][0][1][0] >> 16) : b.a[s][j][1][0] >> shift;
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) acc[s][rb] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a.v, x[rb].v, acc[s][rb], (int)pos, 0, 0);
                }
            } else {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    BtA a0, a1;
                    a0.raw = b.a[s][j][0];
                    a1.raw = b.a[s][j][1];
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) acc[s][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0.v, x[rb].h[0], acc[s][rb], 0, 0, 0);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) acc[s][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1.v, x[rb].h[1], acc[s][rb], 0, 0, 0);
                }
            }
        }
    };
    auto lds_barrier = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    auto steps_of = [&](int u) { return TILE == 128 ? 2 : (Tk - 2 * u < 2 ? Tk - 2 * u : 2); };

    // Two register buffers alternate, unit u + 1 requested before unit u is multiplied.  No load of the loop is conditional
    // (behind a branch the compiler would wait for the loads of either arm), so the last one or two units are written out.
    BtW wa, wb;
    const int n = (u1 - u0 + KG - 1) / KG;   // units per wavefront group: u0 + kg, u0 + kg + KG, ... (the last may not exist)
    auto at = [&](int i) { const int u = u0 + kg + i * KG; return u < u1 ? u : u1 - 1; };
    auto last_steps = [&](int i) { return u0 + kg + i * KG < u1 ? steps_of(u0 + kg + i * KG) : 0; };
    uint32_t ea0 = entry(at(0), 0), ea1 = entry(at(0), 1);
    uint32_t eb0 = entry(at(1), 0), eb1 = entry(at(1), 1);
    load_x(at(0));
    load_w(wa, ea0, ea1);
    store_x(0);
    lds_barrier();
    int i = 0;
    for (; i + 2 < n; i += 2) {
        const uint32_t ec0 = entry(at(i + 2), 0), ec1 = entry(at(i + 2), 1), ed0 = entry(at(i + 3), 0), ed1 = entry(at(i + 3), 1);
        load_x(at(i + 1));
        load_w(wb, eb0, eb1);
        compute(wa, ea0, ea1, 0, 2);
        store_x(1);
        lds_barrier();
        load_x(at(i + 2));
        load_w(wa, ec0, ec1);
        compute(wb, eb0, eb1, 1, 2);
        store_x(0);
        lds_barrier();
        ea0 = ec0; ea1 = ec1; eb0 = ed0; eb1 = ed1;
    }
    if (i + 1 < n) {
        load_x(at(i + 1));
        load_w(wb, eb0, eb1);
        compute(wa, ea0, ea1, 0, 2);
        store_x(1);
        lds_barrier();
        if (const int steps = last_steps(i + 1)) compute(wb, eb0, eb1, 1, steps);
    } else {
        if (const int steps = last_steps(i)) compute(wa, ea0, ea1, 0, steps);
    }
    // the groups' partial sums meet in LDS, added in group order
    if constexpr (KG > 1) {
        __syncthreads();
        bt_f32x4* const red = reinterpret_cast<bt_f32x4*>(lds_all);   // [KG - 1][4 wavefronts][2 RB][64]
        static_assert((KG - 1) * 4 * 2 * RB * 64 * 16 <= KG * 2 * kStage, "the sums fit where X was");
        if (kg > 0)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) red[(((kg - 1) * 4 + w) * 2 * RB + s * RB + rb) * 64 + lane] = acc[s][rb];
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int g = 1; g < KG; ++g)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const bt_f32x4 v = red[(((g - 1) * 4 + w) * 2 * RB + s * RB + rb) * 64 + lane];
                    acc[s][rb][0] += v[0]; acc[s][rb][1] += v[1]; acc[s][rb][2] += v[2]; acc[s][rb][3] += v[3];
                }
    }

    // acc[s][rb][r] = Y^T[n0 + 16 s + 4 q + r][16 rb + col]
    float* dst = SPLIT ? Y + (int64_t)blockIdx.y * rows * N : ybf16 ? reinterpret_cast<float*>(reinterpret_cast<uint16_t*>(Y) + m0 * N) : Y + m0 * N;
    if (live)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                if (16 * rb + col < rows) store4(dst, (int64_t)(16 * rb + col) * N + n0 + 16 * s + 4 * q, acc[s][rb], SPLIT ? 0 : ybf16);
}

template <int TILE, bool SPLIT>
static void launch_batch_t(const GemmArgs& a, const WeightSet& set, int64_t m0, int rows, int split, int ybf16, hipStream_t stream) {
    const dim3 grid((unsigned)set.units, (unsigned)split), block(256 * kBtGroups);
    if (rows <= 16) hipLaunchKernelGGL((batch_kernel<TILE, 1, SPLIT>), grid, block, 0, stream, a.X, m0, rows, a.K, a.Tk, set, ybf16);
    else if (rows <= 32) hipLaunchKernelGGL((batch_kernel<TILE, 2, SPLIT>), grid, block, 0, stream, a.X, m0, rows, a.K, a.Tk, set, ybf16);
    else if (rows <= 48) hipLaunchKernelGGL((batch_kernel<TILE, 3, SPLIT>), grid, block, 0, stream, a.X, m0, rows, a.K, a.Tk, set, ybf16);
    else hipLaunchKernelGGL((batch_kernel<TILE, 4, SPLIT>), grid, block, 0, stream, a.X, m0, rows, a.K, a.Tk, set, ybf16);
}

// Up to 64 rows of X starting at row m0.  set.units / first[] count groups of 128 features, each weight rounded up.  A K split
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
