// The batched-decoding product shared by the bf16 weights (gemm_batch.hip, up to 128 rows of X per launch; it says what bounds the
// kernel) and the 4-bit storage (quant4.hip, up to 64).
#pragma once
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
typedef const PATCH_BT_GLOBAL uint16_t* bt_halves_ptr;

constexpr int kBtFeatures = 128;   // per workgroup: 4 wavefronts x 2 strips
constexpr int kBtUnit = 128;       // columns per unit
// wavefront groups, each taking every kth unit: two up to 64 rows; beyond, the accumulators of 128 rows leave room for one
constexpr int bt_groups(int RB) { return RB > 4 ? 1 : 2; }

__device__ __forceinline__ uint64_t bt_uniform64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// The product for feature group grp of a weight (payload, table, N; `scales` in the 4-bit storage).  Weight = how a wavefront
// holds the weights of a unit.  RB = 16-row blocks of X.  SPLIT: gridDim.y K-chunks, partial sums to a workspace (Y; chunk c
// at c x rows x N).
template <class Weight, int TILE, int RB, bool SPLIT>
__device__ __forceinline__ void batch_body(const uint16_t* __restrict__ X, int64_t m0, int rows, int64_t K, int Tk, bt_bytes_ptr payload,
                                           bt_table_ptr table, bt_halves_ptr scales, float* Y, int64_t N, int grp, int ybf16) {
    constexpr int KG = bt_groups(RB);
    constexpr int kStage = 2 * RB * 16 * 128;   // two steps x rows x 128 bytes
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[KG * 2 * kStage];
    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), kg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    uint8_t* const lds = lds_all + kg * 2 * kStage;
    const int col = lane & 15, q = lane >> 4;
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

    const bt_halves_ptr srow = scales + ((n0 / 16) * Tk * 16 + col);   // (4-bit storage) scale of this lane's row of the first strip, tile 0
    auto entry = [&](int u, int j) -> uint32_t {   // of step j of unit u (past the end: the last tile)
        int t = TILE == 128 ? u : 2 * u + j;
        t = t < Tk ? t : Tk - 1;
        return trow[t];
    };
    typedef typename Weight::template Unit<TILE> Unit;
    auto load_w = [&](Unit& b, uint32_t e0, uint32_t e1, int u) {
        int t0 = TILE == 128 ? u : 2 * u, t1 = TILE == 128 ? u : 2 * u + 1;
        t0 = t0 < Tk ? t0 : Tk - 1;
        t1 = t1 < Tk ? t1 : Tk - 1;
        b.load(payload, srow, Tk, e0, e1, t0, t1, s0, lane);
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
    auto compute = [&](const Unit& b, uint32_t e0, uint32_t e1, int stage, int steps) {
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
                    a.raw = b.operand(s, j, 0);
                    const uint32_t pos = b.positions(s, j, lane);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) acc[s][rb] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a.v, x[rb].v, acc[s][rb], (int)pos, 0, 0);
                }
            } else {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    BtA a0, a1;
                    a0.raw = b.operand(s, j, 0);
                    a1.raw = b.operand(s, j, 1);
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
    Unit wa, wb;
    const int n = (u1 - u0 + KG - 1) / KG;   // units per wavefront group: u0 + kg, u0 + kg + KG, ... (the last may not exist)
    auto at = [&](int i) { const int u = u0 + kg + i * KG; return u < u1 ? u : u1 - 1; };
    auto last_steps = [&](int i) { return u0 + kg + i * KG < u1 ? steps_of(u0 + kg + i * KG) : 0; };
    uint32_t ea0 = entry(at(0), 0), ea1 = entry(at(0), 1);
    uint32_t eb0 = entry(at(1), 0), eb1 = entry(at(1), 1);
    load_x(at(0));
    load_w(wa, ea0, ea1, at(0));
    store_x(0);
    lds_barrier();
    int i = 0;
    for (; i + 2 < n; i += 2) {
        const uint32_t ec0 = entry(at(i + 2), 0), ec1 = entry(at(i + 2), 1), ed0 = entry(at(i + 3), 0), ed1 = entry(at(i + 3), 1);
        load_x(at(i + 1));
        load_w(wb, eb0, eb1, at(i + 1));
        compute(wa, ea0, ea1, 0, 2);
        store_x(1);
        lds_barrier();
        load_x(at(i + 2));
        load_w(wa, ec0, ec1, at(i + 2));
        compute(wb, eb0, eb1, 1, 2);
        store_x(0);
        lds_barrier();
        ea0 = ec0; ea1 = ec1; eb0 = ed0; eb1 = ed1;
    }
    if (i + 1 < n) {
        load_x(at(i + 1));
        load_w(wb, eb0, eb1, at(i + 1));
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

}  // namespace patch
