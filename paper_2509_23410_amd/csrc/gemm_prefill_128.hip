// Prefill-shaped hybrid GEMM in blocks of 256 features x 128 rows (Section 4 / Appendix A of the paper: the product for the prefill input,
// dense and 2:4 tiles mixed inside one launch): the kernel of a few hundred rows, where blocks of 256 rows are too few to fill the chip.
//
// What bounds it: the loop.  A K-step is 32 matrix instructions (dense; 16 sparse) per wavefront of 32 cycles each, and per compute unit 16 KB of X
// and 32 KB (18) of weights from the L2.  Counted on 15360 x 5120, 512 rows (240 workgroups, 70 us at f = 1/2), f = 0 / 1/2 / 1: the matrix pipes are busy 60 / 51 / 41 %
// of a wavefront's life and a compute unit draws 30 / 29 / 29 bytes per clock from the L2, whatever f; wavefronts wait 50 / 42 / 34 % of the time.
// prefill_kernel_areg runs the same block with eight wavefronts of 32 features: each 16 bytes of X read from LDS serve one matrix instruction, two wavefronts of
// a SIMD wait at the same two barriers of every step, and its loads are one step ahead.  Here four wavefronts own 64 features x 128 rows each, so that an X
// operand read from LDS serves two matrix instructions; the weights of two steps are in flight or in use in registers that the asm statements name (v192 -
// v255, two buffers) and the X of three more in four LDS stages (64 KB); and the operands of the next half-step are read between the matrix instructions of
// this one, over the barrier: one barrier per step.  Waits are counted by hand (vmcnt), since loads into LDS and into registers share the counter and the
// compiler would wait for all of them.  64 KB of LDS and at most 256 registers leave room for a second workgroup on the compute unit.
//
// Measured against prefill_kernel_areg, unsplit, f = 1/2, mask tile 128: 4096 x 4096, 128 rows 63.6 -> 52.0 us; 4096 x 8192, 128 rows 123 -> 96 (f = 0
// 144 -> 106, f = 1 107 -> 87); mask tile 64, 4096 x 8192, 128 rows 122 -> 93.  Against what a call with a workspace took before, weights from memory: 5120 x
// 5120, 512 rows in three slices with their sum 44.0 -> 38.1; three of them sharing X 73.1 -> 70.6.  Against the 256-row kernels it gains only while its
// blocks are one round of the chip (see prefill_r128_split).  Tried and slower: areg's eight wavefronts with X in a ring of four stages (52.3 / 99.4 us for
// the first two).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "epilogue.h"
#include "kernels.h"
#include "layout.h"
#include "prefill_parts.h"
#include "tile_order.h"

namespace patch {

constexpr int kRhBN = 256, kRhBM = 128;
constexpr int kRhStage = kRhBM * 128;   // 128 rows of X x 64 columns, swizzled (xs_off)
constexpr int kRhLds = 4 * kRhStage;    // 64 KB: the four X stages

#define PATCH_RH_W(B, FB, I) "v[192+32*" B "+16*" #FB "+4*" #I ":192+32*" B "+16*" #FB "+4*" #I "+3]"
#define PATCH_RH_W0(B, FB, I) "v[192+32*" B "+16*" #FB "+4*" #I "]"
#define PATCH_RH_X(F, C) "v[160+8*" #F "+4*" #C ":160+8*" #F "+4*" #C "+3]"
#define PATCH_RH_XP(F) "v[160+8*" #F ":160+8*" #F "+7]"
#define PATCH_RH_R10(p) "v" #p "0", "v" #p "1", "v" #p "2", "v" #p "3", "v" #p "4", "v" #p "5", "v" #p "6", "v" #p "7", "v" #p "8", "v" #p "9"
#define PATCH_RH_CLOBBER                                                                                                             \
    PATCH_RH_R10(16), PATCH_RH_R10(17), PATCH_RH_R10(18), PATCH_RH_R10(19), PATCH_RH_R10(20), PATCH_RH_R10(21), PATCH_RH_R10(22),     \
        PATCH_RH_R10(23), PATCH_RH_R10(24), "v250", "v251", "v252", "v253", "v254", "v255"

// The four weight loads of half-step U of step buffer B (both 32-feature blocks): t + v[fb][0 / 1]
template <int B, int U>
__device__ __forceinline__ void rh_load(const uint8_t* t, uint32_t v00, uint32_t v01, uint32_t v10, uint32_t v11) {
#define PATCH_RH_LOAD(I0, I1)                                                                                                        \
    asm volatile("global_load_dwordx4 " PATCH_RH_W("%[b]", 0, I0) ", %[v00], %[t]\n\t"                                               \
                 "global_load_dwordx4 " PATCH_RH_W("%[b]", 0, I1) ", %[v01], %[t]\n\t"                                               \
                 "global_load_dwordx4 " PATCH_RH_W("%[b]", 1, I0) ", %[v10], %[t]\n\t"                                               \
                 "global_load_dwordx4 " PATCH_RH_W("%[b]", 1, I1) ", %[v11], %[t]" ::[b] "n"(B), [v00] "v"(v00), [v01] "v"(v01),      \
                 [v10] "v"(v10), [v11] "v"(v11), [t] "s"(t)                                                                          \
                 : "memory", PATCH_RH_CLOBBER)
    if constexpr (U == 0) PATCH_RH_LOAD(0, 1);
    else PATCH_RH_LOAD(2, 3);
#undef PATCH_RH_LOAD
}

// X operands of one position into set F
#define PATCH_RH_READ(F, C, ADDR, OFF) "ds_read_b128 " PATCH_RH_X(F, C) ", %[" #ADDR "] offset:%[" #OFF "]\n\t"
template <int F, int OFF>
__device__ __forceinline__ void rh_fetch(uint32_t r0, uint32_t r1) {
#define PATCH_RH_FETCH(F_)                                                                                                           \
    asm volatile(PATCH_RH_READ(F_, 0, r0, o) PATCH_RH_READ(F_, 1, r1, o)::[r0] "v"(r0), [r1] "v"(r1), [o] "n"(OFF) : "memory", PATCH_RH_CLOBBER)
    if constexpr (F == 0) PATCH_RH_FETCH(0);
    else if constexpr (F == 1) PATCH_RH_FETCH(1);
    else PATCH_RH_FETCH(2);
#undef PATCH_RH_FETCH
}

// Half-step U: four positions (32 rows of X each, operand sets 0 .. 3) against the wavefront's two 32-feature blocks; the reads of the position three
// ahead go into the set of the position before.
#define PATCH_RH_DENSE(P, NF, I0, I1, A0, A1, O)                                                                                     \
    "s_waitcnt lgkmcnt(4)\n\t"                                                                                                       \
    "v_mfma_f32_32x32x16_bf16 %[c0" #P "], " PATCH_RH_W("%[b]", 0, I0) ", " PATCH_RH_X(P, 0) ", %[c0" #P "]\n\t"                     \
    PATCH_RH_READ(NF, 0, A0, O)                                                                                                      \
    "v_mfma_f32_32x32x16_bf16 %[c1" #P "], " PATCH_RH_W("%[b]", 1, I0) ", " PATCH_RH_X(P, 0) ", %[c1" #P "]\n\t"                     \
    PATCH_RH_READ(NF, 1, A1, O)                                                                                                      \
    "v_mfma_f32_32x32x16_bf16 %[c0" #P "], " PATCH_RH_W("%[b]", 0, I1) ", " PATCH_RH_X(P, 1) ", %[c0" #P "]\n\t"                     \
    "v_mfma_f32_32x32x16_bf16 %[c1" #P "], " PATCH_RH_W("%[b]", 1, I1) ", " PATCH_RH_X(P, 1) ", %[c1" #P "]\n\t"
#define PATCH_RH_SPARSE(P, NF, I0, I1, A0, A1, O)                                                                                    \
    "s_waitcnt lgkmcnt(4)\n\t"                                                                                                       \
    "v_smfmac_f32_32x32x32_bf16 %[c0" #P "], " PATCH_RH_W("%[b]", 0, I0) ", " PATCH_RH_XP(P) ", " PATCH_RH_W0("%[b]", 0, I1) "\n\t"   \
    PATCH_RH_READ(NF, 0, A0, O)                                                                                                      \
    "v_smfmac_f32_32x32x32_bf16 %[c1" #P "], " PATCH_RH_W("%[b]", 1, I0) ", " PATCH_RH_XP(P) ", " PATCH_RH_W0("%[b]", 1, I1) "\n\t"   \
    PATCH_RH_READ(NF, 1, A1, O)
// own operands r0, r1 (this half-step's chunks) and n0, n1 (the next one's); offsets h3 (rows 96 .. 127 of this half-step), x0 - x2 (the next one)
#define PATCH_RH_HALF(I0, I1, WAIT, SHIFT, SHC)                                                                                      \
    asm volatile(WAIT "s_cmp_eq_u32 %[sp], 0\n\t"                                                                                    \
                 "s_cbranch_scc1 .Lrhd%=\n\t" SHIFT(I1)                                                                              \
                 PATCH_RH_SPARSE(0, 3, I0, I1, r0, r1, h3) PATCH_RH_SPARSE(1, 0, I0, I1, n0, n1, x0)                                 \
                 PATCH_RH_SPARSE(2, 1, I0, I1, n0, n1, x1) PATCH_RH_SPARSE(3, 2, I0, I1, n0, n1, x2)                                 \
                 "s_branch .Lrhe%=\n"                                                                                                \
                 ".Lrhd%=:\n\t"                                                                                                      \
                 PATCH_RH_DENSE(0, 3, I0, I1, r0, r1, h3) PATCH_RH_DENSE(1, 0, I0, I1, n0, n1, x0)                                   \
                 PATCH_RH_DENSE(2, 1, I0, I1, n0, n1, x1) PATCH_RH_DENSE(3, 2, I0, I1, n0, n1, x2)                                   \
                 ".Lrhe%=:"                                                                                                          \
                 : [c00] "+v"(acc[0][0]), [c01] "+v"(acc[0][1]), [c02] "+v"(acc[0][2]), [c03] "+v"(acc[0][3]), [c10] "+v"(acc[1][0]), \
                   [c11] "+v"(acc[1][1]), [c12] "+v"(acc[1][2]), [c13] "+v"(acc[1][3])                                               \
                 : [b] "n"(B), [sp] "s"(sparse), [sh] SHC(shift), [r0] "v"(r0), [r1] "v"(r1), [n0] "v"(n0), [n1] "v"(n1),             \
                   [h3] "n"(HERE + 12288), [x0] "n"(NEXT), [x1] "n"(NEXT + 4096), [x2] "n"(NEXT + 8192)                              \
                 : "memory", "scc", PATCH_RH_CLOBBER)
#define PATCH_RH_SHIFT(I1)                                                                                                           \
    "v_lshrrev_b32 " PATCH_RH_W0("%[b]", 0, I1) ", %[sh], " PATCH_RH_W0("%[b]", 0, I1) "\n\t"                                        \
    "v_lshrrev_b32 " PATCH_RH_W0("%[b]", 1, I1) ", %[sh], " PATCH_RH_W0("%[b]", 1, I1) "\n\ts_nop 1\n\t"
template <int B, int U, int HERE, int NEXT>
__device__ __forceinline__ void rh_half(f32x16 (&acc)[2][4], int sparse, uint32_t shift, uint32_t r0, uint32_t r1, uint32_t n0, uint32_t n1) {
    if constexpr (U == 0) PATCH_RH_HALF(0, 1, "s_waitcnt vmcnt(16)\n\t", PATCH_RH_SHIFT, "v");
    else PATCH_RH_HALF(2, 3, "", PATCH_RH_SHIFT, "v");
}

template <int TILE, bool SPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void prefill_kernel_r128(
    const uint16_t* __restrict__ X, int64_t M, int64_t K, int Tk_all, int tiles_n, int tiles_m, int t0, int cnt, const WeightSet set, int ybf16) {
    constexpr int KPT = TILE / kStepCols;  // K-steps per tile: 2 or 1
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tr = TILE == 128 ? w >> 1 : w, sh = TILE == 128 ? w & 1 : 0;   // tile row of the block, half of the tile
    // Block -> (n, m): one contiguous run of the order per XCD.  t0 < 0: the launch is a grid of tiles_n x tiles_m blocks.  Otherwise it covers tiles
    // t0 .. of a grid of 256 x 256 tiles, two blocks each.
    const bool tail = t0 >= 0;
    int bid = blockIdx.x;
    {
        const int per = (cnt + 7) / 8;
        const int x = bid & 7, i = bid >> 3;
        const int t = x * per + i;
        bid = (i < per && t < cnt) ? t : -1;
    }
    if (bid < 0) return;
    int bn, bm;
    tile_of(tail ? t0 + (bid >> 1) : bid, tiles_n, tiles_m, bn, bm);
    const int64_t m0 = tail ? (int64_t)bm * 256 + (bid & 1) * kRhBM : (int64_t)bm * kRhBM;
    if (m0 >= M) return;
    // the weight of the set that the feature block belongs to
    uint64_t payload_ = reinterpret_cast<uint64_t>(set.payload[0]), table_ = reinterpret_cast<uint64_t>(set.table[0]), Y_ = reinterpret_cast<uint64_t>(set.Y[0]);
    int64_t N = set.N[0];
    if (set.count > 1) {
        int first = 0;
#pragma unroll
        for (int i = 1; i < kMaxMany; ++i) {
            const bool here = i < set.count && bn >= set.first[i];
            payload_ = here ? reinterpret_cast<uint64_t>(set.payload[i]) : payload_;
            table_ = here ? reinterpret_cast<uint64_t>(set.table[i]) : table_;
            Y_ = here ? reinterpret_cast<uint64_t>(set.Y[i]) : Y_;
            N = here ? set.N[i] : N;
            first = here ? set.first[i] : first;
        }
        bn -= first;
    }
    const uint8_t* const payload = reinterpret_cast<const uint8_t*>(payload_);
    float* const Y = reinterpret_cast<float*>(Y_);
    typedef const __attribute__((address_space(4))) int32_t* pairs_t;
    typedef const __attribute__((address_space(1))) uint32_t* table_t;
    // Mask tile 128: the two tile rows that the packer put together (so that both are 2:4 in as many steps as possible), -1 = no second one.  Mask
    // tile 64: four adjacent tile rows, of which the last block may lack up to three.  A wavefront without a tile row works on another one's
    // weights (valid addresses) and stores nothing.
    bool live;
    int64_t nrow;
    if constexpr (TILE == 128) {
        const pairs_t pairs = reinterpret_cast<pairs_t>(table_) + (N / TILE) * (int64_t)Tk_all;
        const int row0 = pairs[2 * bn], row1 = pairs[2 * bn + 1];
        live = tr == 0 || row1 >= 0;
        nrow = (int64_t)((tr == 0 || row1 < 0) ? row0 : row1) * TILE;
    } else {
        const int64_t n0 = (int64_t)bn * kRhBN;
        live = n0 + w * TILE < N;
        nrow = n0 + (live ? w * TILE : 0);
    }
    const int t_begin = SPLIT ? (int)((int64_t)blockIdx.y * Tk_all / gridDim.y) : 0;
    const int Tk = SPLIT ? (int)((int64_t)(blockIdx.y + 1) * Tk_all / gridDim.y) - t_begin : Tk_all;
    const table_t trow = reinterpret_cast<table_t>(table_) + (nrow / TILE) * Tk_all + t_begin;

    // X tile copy: wavefront w copies the 1 KB pieces w, w + 4, ...
    const uint8_t* xsrc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = (w + 4 * i) * 64 + lane;
        const int m = c >> 3, pp = c & 7, pl = pp ^ ((m >> 1) & 7);
        int64_t row = m0 + m;
        if (row >= M) row = M - 1;
        xsrc[i] = reinterpret_cast<const uint8_t*>(X + row * K + pl * 8 + (int64_t)t_begin * TILE);
    }
    const int i32 = lane & 31, q = lane >> 5;
    // this lane's pieces: strips 4 sh + i32 / 16 and two further on (the second 32-feature block), fragment lane 16 q + i32 % 16
    const int strip = 4 * sh + (i32 >> 4);
    const int flane = 16 * q + (i32 & 15);
    const uint32_t v_val = (uint32_t)(strip * KPT * kSparseFragBytes + flane * 16);
    const uint32_t v_pos = (uint32_t)(sparse_vals_bytes(TILE) + (strip * 64 + flane) * (2 * KPT)) & ~3u;
    const uint32_t v_den = (uint32_t)(strip * KPT * kDenseFragBytes + flane * 16);
    const uint32_t odd_lane = 16u * (flane & 1);   // mask tile 64: which half of a position dword

    f32x16 acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    const int S = Tk * KPT;
    int ent_base = 0;
    uint32_t ent = trow[lane < Tk ? lane : Tk - 1];
    asm volatile("" : "+v"(ent));
    auto entry = [&](int s) __attribute__((always_inline)) {
        const int t = (s < S ? s : S - 1) / KPT;
        if (t >= ent_base + 64) {
            ent_base += 64;
            ent = trow[ent_base + lane < Tk ? ent_base + lane : Tk - 1];
            asm volatile("" : "+v"(ent));   // waited for here, not behind the branch by every step
        }
        return (uint32_t)__builtin_amdgcn_readlane((int)ent, t - ent_base);
    };
    uint32_t eb[4];
    auto load_x = [&](auto buf, int s) __attribute__((always_inline)) {
        constexpr int B = decltype(buf)::value;
        const int sx = s < S ? s : S - 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) g2l16(xsrc[i] + (size_t)sx * 128, lds + B * kRhStage + (w + 4 * i) * 1024);
    };
    auto load_w = [&](auto buf, auto half, int s) __attribute__((always_inline)) {
        constexpr int B = decltype(buf)::value, U = decltype(half)::value;
        if (U == 0) eb[B] = entry(s);
        const uint32_t e = eb[B];
        const bool sp = entry_sparse(e);
        const int j = (s < S ? s : S - 1) % KPT;
        const uint32_t va = sp ? v_val + (uint32_t)(j * kSparseFragBytes + 512 * U) : v_den + (uint32_t)(j * kDenseFragBytes + 1024 * U);
        const uint32_t vb = sp ? v_pos + 64 * KPT * U : va + 512;
        rh_load<B & 1, U>(payload + entry_offset(e), va, vb, va + (sp ? 2 * KPT * kSparseFragBytes : 2 * KPT * kDenseFragBytes),
                          vb + (sp ? 2 * 64 * 2 * KPT : 2 * KPT * kDenseFragBytes));
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)lds;
    const uint32_t xr0 = lds0 + xs_off(i32, q), xr1 = lds0 + xs_off(i32, 2 + q), xr2 = lds0 + xs_off(i32, 4 + q), xr3 = lds0 + xs_off(i32, 6 + q);
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    constexpr std::integral_constant<int, 3> c3{};
    load_x(c0, 0);
    load_x(c1, 1);
    load_w(c0, c0, 0);
    load_w(c0, c1, 0);
    load_x(c2, 2);
    load_w(c1, c0, 1);
    load_w(c1, c1, 1);
    asm volatile("s_waitcnt vmcnt(24)\n\ts_barrier" ::: "memory", PATCH_RH_CLOBBER);
    rh_fetch<0, 0>(xr0, xr1);
    rh_fetch<1, 4096>(xr0, xr1);
    rh_fetch<2, 8192>(xr0, xr1);
    auto step = [&](auto buf, int s) __attribute__((always_inline)) {
        constexpr int B = decltype(buf)::value, kHere = B * kRhStage, kNext = ((B + 1) & 3) * kRhStage;
        const int sp = (int)(eb[B] & 1u);
        const uint32_t shift = KPT == 2 ? 16u * (B & 1) : odd_lane;
        rh_half<B & 1, 0, kHere, kHere>(acc, sp, shift, xr0, xr1, xr2, xr3);
        asm volatile("s_waitcnt vmcnt(12)\n\ts_barrier" ::: "memory", PATCH_RH_CLOBBER);
        load_x(std::integral_constant<int, (B + 3) & 3>{}, s + 3);
        load_w(std::integral_constant<int, (B + 2) & 3>{}, c0, s + 2);
        rh_half<B & 1, 1, kHere, kNext>(acc, sp, shift, xr2, xr3, xr0, xr1);
        load_w(std::integral_constant<int, (B + 2) & 3>{}, c1, s + 2);
    };
    for (int s = 0;; s += 4) {
        step(c0, s);
        if (KPT == 1 && s + 1 >= S) break;
        step(c1, s + 1);
        if (s + 2 >= S) break;
        step(c2, s + 2);
        if (KPT == 1 && s + 3 >= S) break;
        step(c3, s + 3);
        if (s + 4 >= S) break;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory", PATCH_RH_CLOBBER);
    // acc[a][b][i]: feature nrow + 64 sh + 32 a + 8 (i/4) + 4 q + i%4, row m0 + 32 b + i32.  The X stages are free once every wavefront has
    // left the loop.
    __syncthreads();
    if (live) {
        // (a slot of 256 x 256 floats per tile and slice, a part of the workspace per slice, or Y)
        const bool slots = SPLIT && tail;
        const int64_t stride = slots ? 256 : N;
        const int64_t at = slots ? (((int64_t)(bid >> 1) * gridDim.y + blockIdx.y) * 256 + (bid & 1) * kRhBM) * 256 + 64 * w
                                 : (SPLIT ? (int64_t)blockIdx.y * M * N : 0) + m0 * N + nrow + 64 * sh;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                store_block_rows(lds + w * 4096, acc[a][b], lane, Y, at + 32 * b * stride + 32 * a, stride, M - (m0 + 32 * b), SPLIT ? 0 : ybf16);
    }
}

void launch_prefill_r128(const GemmArgs& a, const WeightSet& set, int split, hipStream_t stream) {
    const int tiles_m = (int)((a.M + kRhBM - 1) / kRhBM), nblk = set.units * tiles_m, grid = ((nblk + 7) / 8) * 8;
    if (split < 2) {
        const auto kernel = a.tile == 128 ? &prefill_kernel_r128<128, false> : &prefill_kernel_r128<64, false>;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), kRhLds, stream, a.X, a.M, a.K, a.Tk, set.units, tiles_m, -1, nblk, set, a.ybf16);
        return;
    }
    WeightSet part = set;
    WrReduceSet red = {};
    size_t off = 0;
    for (int i = 0; i < set.count; ++i) {
        part.Y[i] = a.ws + off;
        red.ws[i] = a.ws + off;
        red.Y[i] = set.Y[i];
        red.n4[i] = (size_t)a.M * (size_t)set.N[i] / 4;
        off += (size_t)split * (size_t)a.M * (size_t)set.N[i];
    }
    const auto kernel = a.tile == 128 ? &prefill_kernel_r128<128, true> : &prefill_kernel_r128<64, true>;
    hipLaunchKernelGGL(kernel, dim3(grid, split), dim3(256), kRhLds, stream, a.X, a.M, a.K, a.Tk, set.units, tiles_m, -1, nblk, part, 0);
    if (set.count == 1) wr_reduce(a.ws, red.n4[0], split, set.Y[0], a.ybf16, stream);
    else wr_reduce_set(red, set.count, split, a.ybf16, stream);
}

void launch_prefill_r128_tail(const GemmArgs& a, const WeightSet& set, int tiles_m, int t0, int tail, int slices, hipStream_t stream) {
    const dim3 grid((unsigned)((2 * tail + 7) / 8 * 8), (unsigned)slices);
    const auto kernel = slices > 1 ? a.tile == 128 ? &prefill_kernel_r128<128, true> : &prefill_kernel_r128<64, true>
                                   : a.tile == 128 ? &prefill_kernel_r128<128, false> : &prefill_kernel_r128<64, false>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), kRhLds, stream, a.X, a.M, a.K, a.Tk, set.units, tiles_m, t0, 2 * tail, set, a.ybf16);
}

}  // namespace patch
