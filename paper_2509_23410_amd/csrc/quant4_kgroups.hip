// Prefill-shaped product from the 4-bit storage with K divided between two groups of wavefronts of a workgroup (layout and
// rounding: quant4.hip; Section 5.2 of the paper).
//
// Workgroup = 256 features x 128 rows of X, 8 wavefronts.  Wavefronts 0 - 3 (group 0) own 64 features x all 128 rows each and take the even 64-column
// K-steps, wavefronts 4 - 7 the same features and the odd ones; the two halves meet in LDS at the end (group 0's sum + group 1's: a fixed order).
// Why: prefill4_kernel's wavefronts own 32 features, so that each K-step of X is read from LDS eight times, and each step runs in turn - convert,
// read X, multiply, wait for the loads issued a step ago - on wavefronts that a barrier keeps in line.  Here X is read four times, two wavefronts
// share a SIMD at different K-steps, the conversion of the next operands stands between the matrix instructions of the present ones, codes are
// requested three steps and X three units (of two K-steps) ahead and counted, and one barrier joins two K-steps.  Cycles a K-step, one
// workgroup, cache-resident, f = 0 / 1/2 / 1: 1365 / 1285 / 1066, prefill4_kernel 1900 and more; 11008 x 4096, 500 rows, f = 0 / 1/2 / 1 66.2 / 59.9 / 49.0 ->
// 53.5 / 48.2 / 41.0 us, mask tile 64 67.2 -> 48.5.
// What bounds it: a SIMD's two wavefronts issue about 490 (2:4) or 670 (dense) instructions a unit, and its matrix instructions take 1024 / 2048
// cycles.  Counted on 11008 x 4096, 500 rows, f = 0 / 1/2 / 1: matrix pipes busy 63 / 50 / 38 % of a wavefront's life, vector instructions issued in
// 57 / 48 / 41 % of it, wavefronts waiting 35 / 33 / 36 %; a compute unit draws 17 - 19 bytes per clock from the L2, which sends prefill_kernel_r128 29.
// Measured and not taken: a unit as one branch-free statement per tile type (1.02 - 1.05 times as long), a barrier every two units (1.07), 16-bit
// position loads that need no shift (1.02 - 1.03), operands converted in one piece between phases (1.2 - 1.3).  A wavefront lowers its priority from
// phase to phase, so that of two that share a SIMD the one behind goes first (dense steps 4 % shorter).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "epilogue.h"
#include "layout.h"
#include "prefill_parts.h"
#include "quant4_layout.h"
#include "tile_order.h"

namespace patch {

constexpr int kKgBN = 256, kKgBM = 128;
constexpr int kKgStep = kKgBM * 128;       // X of one K-step: 128 rows x 64 columns, swizzled (xs_off)
constexpr int kKgLds = 4 * 2 * kKgStep;    // 128 KB: four stages of two K-steps

typedef const __attribute__((address_space(1))) uint32_t* kg_g4_t;

// Registers by name: loads into them are counted, not tracked, and they live across statements, so every statement declares them all clobbered and the
// compiler's own values stay below v161 until the output stage (tests/test_prefill_registers.py).  Buffer B = 0 .. 2 (units in rotation), 32-feature block FB, half-step U, 32-row
// block R:
//   v161 - v165                  temporaries of the conversion
//   v[166 + 8 FB : + 7]          weight operands of the half-step being multiplied or the next one: first four, second four (dense only)
//   v[182 + 8 R : + 7]           X operands of 32 rows and a half-step
//   v[214 + 14 B + 4 FB : + 3]   codes: dense (first operand of half-steps 0 and 1, second operand of 0 and 1), 2:4 (half-step 0, -, half-step 1, - until kg_ready)
//   v[222 + 14 B + 2 FB + U]     position words
//   v[226 + 14 B + FB]           scale of the lane's row (16 bits; from kg_ready on 16 times its value)
#define PATCH_KG_C(B, FB, I) "v[214+14*" B "+4*" FB "+" I "]"
#define PATCH_KG_CC(B, FB, I) "v[214+14*" B "+4*" #FB "+" #I ":214+14*" B "+4*" #FB "+" #I "+1]"
#define PATCH_KG_P(B, FB, U) "v[222+14*" B "+2*" FB "+" U "]"
#define PATCH_KG_S(B, FB) "v[226+14*" B "+" FB "]"
#define PATCH_KG_H(FB, I) "v[166+8*" FB "+" #I "]"
#define PATCH_KG_HA(FB) "v[166+8*" FB ":166+8*" FB "+3]"
#define PATCH_KG_HB(FB) "v[170+8*" FB ":170+8*" FB "+3]"
#define PATCH_KG_X(R, C) "v[182+8*" #R "+4*" #C ":182+8*" #R "+4*" #C "+3]"
#define PATCH_KG_XP(R) "v[182+8*" #R ":182+8*" #R "+7]"
#define PATCH_KG_R10(p) "v" #p "0", "v" #p "1", "v" #p "2", "v" #p "3", "v" #p "4", "v" #p "5", "v" #p "6", "v" #p "7", "v" #p "8", "v" #p "9"
#define PATCH_KG_CLOBBER                                                                                                            \
    "v161", "v162", "v163", "v164", "v165", "v166", "v167", "v168", "v169", PATCH_KG_R10(17), PATCH_KG_R10(18), PATCH_KG_R10(19),    \
        PATCH_KG_R10(20), PATCH_KG_R10(21), PATCH_KG_R10(22), PATCH_KG_R10(23), PATCH_KG_R10(24), "v250", "v251", "v252", "v253", "v254", "v255"

// Four pieces of a K-step's X (1 KB each, 4 KB apart), global -> LDS: x + v[i] to l + 4096 i
__device__ __forceinline__ void kg_load_x(const uint8_t* x, const uint32_t (&v)[4], uint32_t l) {
    asm volatile("s_mov_b32 m0, %[l0]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[v0], %[x]\n\t"
                 "s_mov_b32 m0, %[l1]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[v1], %[x]\n\t"
                 "s_mov_b32 m0, %[l2]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[v2], %[x]\n\t"
                 "s_mov_b32 m0, %[l3]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[v3], %[x]" ::[l0] "s"(l), [l1] "s"(l + 4096), [l2] "s"(l + 8192),
                 [l3] "s"(l + 12288), [v0] "v"(v[0]), [v1] "v"(v[1]), [v2] "v"(v[2]), [v3] "v"(v[3]), [x] "s"(x)
                 : "memory", PATCH_KG_CLOBBER);
}

// Loads of a K-step into buffer B: codes of the two 32-feature blocks (two 8-byte pieces each), their scales and, of a 2:4 tile, their position words
template <int B, int KPT>
__device__ __forceinline__ void kg_load(const uint8_t* t, uint32_t v00, uint32_t v01, uint32_t v10, uint32_t v11, uint32_t vp, const uint16_t* sc, uint32_t vs0,
                                        uint32_t vs1, bool sparse) {
    asm volatile("global_load_dwordx2 " PATCH_KG_CC("%[b]", 0, 0) ", %[v00], %[t]\n\t"
                 "global_load_dwordx2 " PATCH_KG_CC("%[b]", 0, 2) ", %[v01], %[t]\n\t"
                 "global_load_dwordx2 " PATCH_KG_CC("%[b]", 1, 0) ", %[v10], %[t]\n\t"
                 "global_load_dwordx2 " PATCH_KG_CC("%[b]", 1, 2) ", %[v11], %[t]\n\t"
                 "global_load_ushort " PATCH_KG_S("%[b]", "0") ", %[vs0], %[sc]\n\t"
                 "global_load_ushort " PATCH_KG_S("%[b]", "1") ", %[vs1], %[sc]" ::[b] "n"(B), [v00] "v"(v00), [v01] "v"(v01), [v10] "v"(v10),
                 [v11] "v"(v11), [t] "s"(t), [sc] "s"(sc), [vs0] "v"(vs0), [vs1] "v"(vs1)
                 : "memory", PATCH_KG_CLOBBER);
#define PATCH_KG_POSITIONS(OP, O01, O10, O11)                                                                                       \
    asm volatile(OP " " PATCH_KG_P("%[b]", "0", "0") ", %[vp], %[t]\n\t" OP " " PATCH_KG_P("%[b]", "0", "1") ", %[vp], %[t] offset:" O01 "\n\t" \
                 OP " " PATCH_KG_P("%[b]", "1", "0") ", %[vp], %[t] offset:" O10 "\n\t" OP " " PATCH_KG_P("%[b]", "1", "1") ", %[vp], %[t] offset:" O11 \
                 ::[b] "n"(B), [vp] "v"(vp), [t] "s"(t) : "memory", PATCH_KG_CLOBBER)
    if (!sparse) return;
    if constexpr (KPT == 2) PATCH_KG_POSITIONS("global_load_dword", "128", "512", "640");
    else PATCH_KG_POSITIONS("global_load_ushort", "64", "256", "320");
#undef PATCH_KG_POSITIONS
}

// Before the first use of a K-step's codes: scales to 16 s as floats; of a 2:4 K-step the codes of half-step 1 (the second piece) to where a dense
// one has them and the position words down by `shift` (mask tile 128: both K-steps of the tile share a dword)
template <int B>
__device__ __forceinline__ void kg_ready(int sparse, int shift) {
    asm volatile("v_lshlrev_b32 " PATCH_KG_S("%[b]", "0") ", 16, " PATCH_KG_S("%[b]", "0") "\n\t"
                 "v_lshlrev_b32 " PATCH_KG_S("%[b]", "1") ", 16, " PATCH_KG_S("%[b]", "1") "\n\t"
                 "v_mul_f32 " PATCH_KG_S("%[b]", "0") ", 0x41800000, " PATCH_KG_S("%[b]", "0") "\n\t"
                 "v_mul_f32 " PATCH_KG_S("%[b]", "1") ", 0x41800000, " PATCH_KG_S("%[b]", "1") "\n\t"
                 "s_cmp_eq_u32 %[sp], 0\n\ts_cbranch_scc1 .Lkgp%=\n\t"
                 "v_mov_b32 " PATCH_KG_C("%[b]", "0", "1") ", " PATCH_KG_C("%[b]", "0", "2") "\n\t"
                 "v_mov_b32 " PATCH_KG_C("%[b]", "1", "1") ", " PATCH_KG_C("%[b]", "1", "2") "\n\t"
                 "v_lshrrev_b32 " PATCH_KG_P("%[b]", "0", "0") ", %[sh], " PATCH_KG_P("%[b]", "0", "0") "\n\t"
                 "v_lshrrev_b32 " PATCH_KG_P("%[b]", "0", "1") ", %[sh], " PATCH_KG_P("%[b]", "0", "1") "\n\t"
                 "v_lshrrev_b32 " PATCH_KG_P("%[b]", "1", "0") ", %[sh], " PATCH_KG_P("%[b]", "1", "0") "\n\t"
                 "v_lshrrev_b32 " PATCH_KG_P("%[b]", "1", "1") ", %[sh], " PATCH_KG_P("%[b]", "1", "1") "\n"
                 ".Lkgp%=:" ::[b] "n"(B), [sp] "s"(sparse), [sh] "s"(shift)
                 : "memory", "scc", PATCH_KG_CLOBBER);
}

// Dequantization of one code register C with 16 s in S: four operand registers, in steps of one (q4_dequant8).  Temporaries v161 - v165.
#define PATCH_KG_CVT(dst, src, byte) "v_cvt_off_f32_i4_sdwa " dst ", " src " dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #byte "\n\t"
#define PATCH_KG_V0(C) "v_lshrrev_b32 v161, 4, " C "\n\t"
#define PATCH_KG_V1(C, S, OUT, P, T0, T1)                                                                                            \
    PATCH_KG_CVT(T0, C, P) PATCH_KG_CVT(T1, "v161", P) "v_mul_f32 " T0 ", " S ", " T0 "\n\tv_mul_f32 " T1 ", " S ", " T1 "\n\t"        \
    "v_cvt_pk_bf16_f32 " OUT ", " T0 ", " T1 "\n\t"
// first (A) or second (B) operand of 32-feature block FB (a digit in quotes) from code register I of buffer NB, in four parts
#define PATCH_KG_DA(P, T0, T1) PATCH_KG_V1(PATCH_KG_C("%[nb]", "%[nf]", "%[ni]"), PATCH_KG_S("%[nb]", "%[nf]"), PATCH_KG_H("%[nf]", P), P, T0, T1)
#define PATCH_KG_DB(P, T0, T1) PATCH_KG_V1(PATCH_KG_C("%[nb]", "%[nf]", "%[ni]+2"), PATCH_KG_S("%[nb]", "%[nf]"), PATCH_KG_H("%[nf]", P+4), P, T0, T1)
#define PATCH_KG_A0 PATCH_KG_V0(PATCH_KG_C("%[nb]", "%[nf]", "%[ni]")) PATCH_KG_DA(0, "v162", "v163")
#define PATCH_KG_A1 PATCH_KG_DA(1, "v164", "v165")
#define PATCH_KG_A2 PATCH_KG_DA(2, "v162", "v163")
#define PATCH_KG_A3 PATCH_KG_DA(3, "v164", "v165")
#define PATCH_KG_B0 PATCH_KG_V0(PATCH_KG_C("%[nb]", "%[nf]", "%[ni]+2")) PATCH_KG_DB(0, "v162", "v163")
#define PATCH_KG_B1 PATCH_KG_DB(1, "v164", "v165")
#define PATCH_KG_B2 PATCH_KG_DB(2, "v162", "v163")
#define PATCH_KG_B3 PATCH_KG_DB(3, "v164", "v165")

// The second operand of a dense step / both operands, on their own
template <int NB, int NF, int NI, bool BOTH>
__device__ __forceinline__ void kg_operands(int sparse) {
    if constexpr (BOTH) asm volatile(PATCH_KG_A0 PATCH_KG_A1 PATCH_KG_A2 PATCH_KG_A3 ::[nb] "n"(NB), [nf] "n"(NF), [ni] "n"(NI) : PATCH_KG_CLOBBER);
    asm volatile("s_cmp_lg_u32 %[sp], 0\n\ts_cbranch_scc1 .Lkgo%=\n\t" PATCH_KG_B0 PATCH_KG_B1 PATCH_KG_B2 PATCH_KG_B3 ".Lkgo%=:" ::[nb] "n"(NB), [nf] "n"(NF),
                 [ni] "n"(NI), [sp] "s"(sparse)
                 : "scc", PATCH_KG_CLOBBER);
}

// A phase: 32-feature block FB of half-step U against the four 32-row blocks, and between its matrix instructions the conversion of the operands that
// the next phase multiplies (32-feature block 1 - FB, half-step NI, buffer NB).  FB 0 waits for the X operands, FB 1 requests the next half-step's (lane
// addresses r0 / r1), each set after its last use.
#define PATCH_KG_W(N) "s_waitcnt lgkmcnt(" #N ")\n\t"
#define PATCH_KG_LO(R) "v_mfma_f32_32x32x16_bf16 %[c" #R "], " PATCH_KG_HA("%[fb]") ", " PATCH_KG_X(R, 0) ", %[c" #R "]\n\t"
#define PATCH_KG_HI(R) "v_mfma_f32_32x32x16_bf16 %[c" #R "], " PATCH_KG_HB("%[fb]") ", " PATCH_KG_X(R, 1) ", %[c" #R "]\n\t"
#define PATCH_KG_SP(R) "v_smfmac_f32_32x32x32_bf16 %[c" #R "], " PATCH_KG_HA("%[fb]") ", " PATCH_KG_XP(R) ", " PATCH_KG_P("%[b]", "%[fb]", "%[u]") "\n\t"
#define PATCH_KG_RD(R) "ds_read_b128 " PATCH_KG_X(R, 0) ", %[r0] offset:4096*" #R "\n\tds_read_b128 " PATCH_KG_X(R, 1) ", %[r1] offset:4096*" #R "\n\t"
template <int B, int FB, int U>
__device__ __forceinline__ void kg_phase(f32x16 (&c)[4], int sparse, uint32_t r0, uint32_t r1) {
    constexpr int NB = FB == 1 && U == 1 ? (B + 1) % 3 : B, NF = 1 - FB, NI = FB == 0 ? U : 1 - U;
#define PATCH_KG_PHASE(D, S)                                                                                                        \
    asm volatile("s_cmp_eq_u32 %[sp], 0\n\ts_cbranch_scc1 .Lkgd%=\n\t" S "s_branch .Lkge%=\n.Lkgd%=:\n\t" D ".Lkge%=:"              \
                 : [c0] "+v"(c[0]), [c1] "+v"(c[1]), [c2] "+v"(c[2]), [c3] "+v"(c[3])                                                \
                 : [b] "n"(B), [fb] "n"(FB), [u] "n"(U), [nb] "n"(NB), [nf] "n"(NF), [ni] "n"(NI), [sp] "s"(sparse), [r0] "v"(r0), [r1] "v"(r1) \
                 : "memory", "scc", PATCH_KG_CLOBBER)
    if constexpr (FB == 0 && U == 0) __builtin_amdgcn_s_setprio(3);
    else if constexpr (U == 0) __builtin_amdgcn_s_setprio(2);
    else if constexpr (FB == 0) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
    if constexpr (FB == 0)
        PATCH_KG_PHASE(PATCH_KG_W(6) PATCH_KG_LO(0) PATCH_KG_A0 PATCH_KG_W(4) PATCH_KG_LO(1) PATCH_KG_A1 PATCH_KG_W(2) PATCH_KG_LO(2) PATCH_KG_A2
                       PATCH_KG_W(0) PATCH_KG_LO(3) PATCH_KG_A3 PATCH_KG_HI(0) PATCH_KG_B0 PATCH_KG_HI(1) PATCH_KG_B1 PATCH_KG_HI(2) PATCH_KG_B2
                       PATCH_KG_HI(3) PATCH_KG_B3,
                       PATCH_KG_W(6) PATCH_KG_SP(0) PATCH_KG_A0 PATCH_KG_W(4) PATCH_KG_SP(1) PATCH_KG_A1 PATCH_KG_W(2) PATCH_KG_SP(2) PATCH_KG_A2
                       PATCH_KG_W(0) PATCH_KG_SP(3) PATCH_KG_A3);
    else if constexpr (U == 0)
        PATCH_KG_PHASE(PATCH_KG_LO(0) PATCH_KG_A0 PATCH_KG_LO(1) PATCH_KG_A1 PATCH_KG_LO(2) PATCH_KG_A2 PATCH_KG_LO(3) PATCH_KG_A3
                       PATCH_KG_HI(0) PATCH_KG_RD(0) PATCH_KG_B0 PATCH_KG_HI(1) PATCH_KG_RD(1) PATCH_KG_B1 PATCH_KG_HI(2) PATCH_KG_RD(2) PATCH_KG_B2
                       PATCH_KG_HI(3) PATCH_KG_RD(3) PATCH_KG_B3,
                       PATCH_KG_SP(0) PATCH_KG_RD(0) PATCH_KG_A0 PATCH_KG_SP(1) PATCH_KG_RD(1) PATCH_KG_A1 PATCH_KG_SP(2) PATCH_KG_RD(2) PATCH_KG_A2
                       PATCH_KG_SP(3) PATCH_KG_RD(3) PATCH_KG_A3);
    else   // the next operands are another tile's: the first one here, the second, if it is dense, by kg_operands
        PATCH_KG_PHASE(PATCH_KG_LO(0) PATCH_KG_A0 PATCH_KG_LO(1) PATCH_KG_A1 PATCH_KG_LO(2) PATCH_KG_A2 PATCH_KG_LO(3) PATCH_KG_A3
                       PATCH_KG_HI(0) PATCH_KG_RD(0) PATCH_KG_HI(1) PATCH_KG_RD(1) PATCH_KG_HI(2) PATCH_KG_RD(2) PATCH_KG_HI(3) PATCH_KG_RD(3),
                       PATCH_KG_SP(0) PATCH_KG_RD(0) PATCH_KG_A0 PATCH_KG_SP(1) PATCH_KG_RD(1) PATCH_KG_A1 PATCH_KG_SP(2) PATCH_KG_RD(2) PATCH_KG_A2
                       PATCH_KG_SP(3) PATCH_KG_RD(3) PATCH_KG_A3);
#undef PATCH_KG_PHASE
}
__device__ __forceinline__ void kg_fetch(uint32_t r0, uint32_t r1) {
    asm volatile(PATCH_KG_RD(0) PATCH_KG_RD(1) PATCH_KG_RD(2) PATCH_KG_RD(3)::[r0] "v"(r0), [r1] "v"(r1) : "memory", PATCH_KG_CLOBBER);
}

template <int TILE, bool SPLIT>
__global__ __launch_bounds__(512) void prefill4_kgroups_kernel(const uint16_t* __restrict__ X, int64_t M, int64_t N, int64_t K,
                                                               const uint8_t* __restrict__ payload, const uint16_t* __restrict__ scales,
                                                               const uint32_t* __restrict__ table, int Tk_all, int tiles_n, int tiles_m, int t0,
                                                               int cnt, int slots, float* __restrict__ Y) {
    constexpr int KPT = TILE / kStepCols;      // K-steps per tile: 2 or 1
    extern __shared__ __attribute__((aligned(256))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = w >> 2, fw = w & 3;                                        // K group, 64-feature group
    const int tr = TILE == 128 ? fw >> 1 : fw, sh = TILE == 128 ? fw & 1 : 0;   // tile row of the block, half of the tile
    // blocks t0 .. t0 + cnt - 1 of the order, one contiguous run of it per XCD
    int bid = blockIdx.x;
    {
        const int per = (cnt + 7) / 8;
        const int x = bid & 7, i = bid >> 3;
        const int t = x * per + i;
        bid = (i < per && t < cnt) ? t : -1;
    }
    if (bid < 0) return;
    int bn, bm;
    tile_of(t0 + bid, tiles_n, tiles_m, bn, bm);
    const int64_t n0 = (int64_t)bn * kKgBN, m0 = (int64_t)bm * kKgBM;
    // N is a multiple of the tile, not necessarily of 256: a wavefront of a missing tile row works on the last live one's
    // weights (valid addresses) and stores nothing
    const int rows_here = (int)((N - n0) / TILE) < kKgBN / TILE ? (int)((N - n0) / TILE) : kKgBN / TILE;
    const int64_t trow_n = n0 / TILE + (tr < rows_here ? tr : rows_here - 1);
    const int t_begin = SPLIT ? (int)((int64_t)blockIdx.y * Tk_all / gridDim.y) : 0;
    const int Tk = SPLIT ? (int)((int64_t)(blockIdx.y + 1) * Tk_all / gridDim.y) - t_begin : Tk_all;
    const kg_g4_t trow = (kg_g4_t)(table + trow_n * Tk_all + t_begin);

    // X copy: the group's four wavefronts copy its K-step in 1 KB pieces fw, fw + 4, ...: bytes from row m0 and the slice's first column
    uint32_t xoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = (fw + 4 * i) * 64 + lane;
        const int m = c >> 3, pp = c & 7, pl = pp ^ ((m >> 1) & 7);
        const int64_t row = m0 + m < M ? m : M - 1 - m0;   // rows past M: the last one, not stored
        xoff[i] = (uint32_t)((row * K + pl * 8) * 2);
    }
    const uint8_t* const xbase = reinterpret_cast<const uint8_t*>(X + m0 * K + (int64_t)t_begin * TILE);
    const int i32 = lane & 31, q = lane >> 5;
    // this lane's pieces: strips 4 sh + i32 / 16 and (second 32-feature block) two further on, fragment lanes fl and fl + 32
    const int strip = 4 * sh + (i32 >> 4), fl = 16 * q + (i32 & 15);
    const uint32_t v_den = (uint32_t)((strip * KPT + (KPT == 2 ? g : 0)) * 512 + fl * 8), v_spa = (uint32_t)((strip * KPT + (KPT == 2 ? g : 0)) * 256 + fl * 4);
    const uint32_t v_pos = (uint32_t)(q4_sparse_codes(TILE) + (strip * 64 + fl) * (2 * KPT));
    const uint16_t* const sc = scales + q4_scale_index(trow_n * (TILE / 16) + 4 * sh, Tk_all, t_begin, 0);
    const uint32_t v_sc = (uint32_t)((i32 >> 4) * Tk_all * 16 + (i32 & 15)) * 2;

    f32x16 acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    const int U = KPT == 2 ? Tk : (Tk + 1) / 2;   // units of two K-steps
    int ent_base = 0;
    uint32_t ent = trow[lane < Tk ? lane : Tk - 1];   // table entries of 64 tiles, one per lane
    asm volatile("" : "+v"(ent));
    auto tile_at = [&](int n) __attribute__((always_inline)) {   // tile of this group's K-step of unit n
        const int t = KPT == 2 ? n : 2 * n + g;
        return t < Tk ? t : Tk - 1;
    };
    auto entry = [&](int n) __attribute__((always_inline)) {
        const int t = tile_at(n);
        if (t >= ent_base + 64) {
            ent_base += 64;
            ent = trow[ent_base + lane < Tk ? ent_base + lane : Tk - 1];
            asm volatile("" : "+v"(ent));   // waited for here, not behind the branch by every unit
        }
        return (uint32_t)__builtin_amdgcn_readlane((int)ent, t - ent_base);
    };
    uint32_t eb[3];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)lds;
    const uint32_t lds_x = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + g * kKgStep + fw * 1024));
    auto load_x = [&](int n) __attribute__((always_inline)) {
        const int t = KPT == 2 ? 2 * (n < U ? n : U - 1) + g : tile_at(n);   // K-step
        kg_load_x(xbase + (size_t)t * 128, xoff, lds_x + (uint32_t)(n & 3) * (2 * kKgStep));
    };
    auto load_w = [&](auto buf, int n) __attribute__((always_inline)) {
        constexpr int B = decltype(buf)::value;
        const uint32_t e = eb[B] = entry(n);
        const bool sp = entry_sparse(e);
        const uint32_t v = sp ? v_spa : v_den, gap = sp ? 128 : 256, next = sp ? 2 * KPT * 256 : 2 * KPT * 512;
        kg_load<B, KPT>(payload + entry_offset(e), v, v + gap, v + next, v + next + gap, v_pos, sc + (size_t)tile_at(n) * 16, v_sc, v_sc + 64 * Tk_all, sp);
    };
    const uint32_t xr = lds0 + g * kKgStep + xs_off(i32, q);   // chunk 2 c + q of the row is at xr ^ 32 c
    auto at = [&](int n, int c) __attribute__((always_inline)) { return (xr ^ (32u * c)) + (uint32_t)(n & 3) * (2 * kKgStep); };
    constexpr std::integral_constant<int, 0> k0{};
    constexpr std::integral_constant<int, 1> k1{};
    constexpr std::integral_constant<int, 2> k2{};
    load_x(0); load_w(k0, 0);
    load_x(1); load_w(k1, 1);
    load_x(2); load_w(k2, 2);
    asm volatile("s_waitcnt vmcnt(20)\n\ts_barrier" ::: "memory", PATCH_KG_CLOBBER);
    kg_ready<0>((int)(eb[0] & 1u), KPT == 2 ? 16 * g : 0);
    kg_operands<0, 0, 0, true>((int)(eb[0] & 1u));
    kg_fetch(at(0, 0), at(0, 1));
    auto unit = [&](auto buf, int n) __attribute__((always_inline)) {
        constexpr int B = decltype(buf)::value, BN = (B + 1) % 3;
        const int sp = __builtin_amdgcn_readfirstlane((int)(eb[B] & 1u)), spn = __builtin_amdgcn_readfirstlane((int)(eb[BN] & 1u));
        const bool here = KPT == 2 || 2 * n + g < Tk;   // the last unit of an odd number of tiles lacks its second K-step
        if (here) {
            kg_phase<B, 0, 0>(acc[0], sp, 0u, 0u);
            kg_phase<B, 1, 0>(acc[1], sp, at(n, 2), at(n, 3));
            kg_phase<B, 0, 1>(acc[0], sp, 0u, 0u);
        }
        // X(n + 1) and the weights of unit n + 1 have landed (issued since: X and weights of unit n + 2, ten loads or, with position words, fourteen); past
        // the barrier all of X(n + 1) is visible and every read of X(n - 1), whose stage X(n + 3) takes, has completed
        asm volatile("s_waitcnt vmcnt(10)\n\ts_barrier" ::: "memory", PATCH_KG_CLOBBER);
        load_x(n + 3);
        kg_ready<BN>(spn, KPT == 2 ? 16 * g : 0);
        if (here) {
            kg_phase<B, 1, 1>(acc[1], sp, at(n + 1, 0), at(n + 1, 1));
            kg_operands<BN, 0, 0, false>(spn);
        }
        load_w(buf, n + 3);
    };
    for (int n = 0;; n += 3) {
        unit(k0, n);
        if (n + 1 >= U) break;
        unit(k1, n + 1);
        if (n + 2 >= U) break;
        unit(k2, n + 2);
        if (n + 3 >= U) break;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory", PATCH_KG_CLOBBER);
    // acc[a][b][i]: feature 64 fw + 32 a + 8 (i/4) + 4 q + i%4 of the block, row 32 b + i32: the sums over this group's K-steps.  The wavefronts fw of both
    // groups exchange halves through LDS - group 0 finishes the upper 64 rows, group 1 the lower - and store them (store_block_rows).
    __syncthreads();
    uint8_t* const mine = lds + w * 16384;
    uint8_t* const other = lds + (w ^ 4) * 16384;
    auto put = [&](int k, const f32x16& v) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<f32x4*>(other + k * 4096 + r * 1024 + lane * 16) = f32x4{v[4 * r], v[4 * r + 1], v[4 * r + 2], v[4 * r + 3]};
    };
    auto finish = [&](f32x16& v, int k, int a, int b) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const f32x4 o = *reinterpret_cast<const f32x4*>(mine + k * 4096 + r * 1024 + lane * 16);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[4 * r + i] += o[i];
        }
        // to Y, to a part of the workspace per slice, or to a slot of 128 x 256 floats per block and slice
        const int64_t stride = SPLIT && slots ? kKgBN : N;
        const int64_t at = SPLIT && slots ? ((int64_t)bid * gridDim.y + blockIdx.y) * (kKgBM * kKgBN) : (SPLIT ? (int64_t)blockIdx.y * M * N : 0) + m0 * N + n0;
        if (tr < rows_here) store_block_rows(mine + k * 4096, v, lane, Y, at + 32 * b * stride + 64 * fw + 32 * a, stride, M - (m0 + 32 * b), 0);
    };
    if (g == 0) {
        put(0, acc[0][2]); put(1, acc[0][3]); put(2, acc[1][2]); put(3, acc[1][3]);
    } else {
        put(0, acc[0][0]); put(1, acc[0][1]); put(2, acc[1][0]); put(3, acc[1][1]);
    }
    __syncthreads();
    if (g == 0) {
        finish(acc[0][0], 0, 0, 0); finish(acc[0][1], 1, 0, 1); finish(acc[1][0], 2, 1, 0); finish(acc[1][1], 3, 1, 1);
    } else {
        finish(acc[0][2], 0, 0, 2); finish(acc[0][3], 1, 0, 3); finish(acc[1][2], 2, 1, 2); finish(acc[1][3], 3, 1, 3);
    }
}

static hipError_t kg_grant(decltype(&prefill4_kgroups_kernel<128, false>) kernel) {   // more LDS than a launch gets without asking
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kKgLds);
}

// Sum of the slots of the last `cnt` blocks (slice 0 first) into Y.  Workgroup = 16 rows of a block; thread = 4 x 4 features of one row.
__global__ __launch_bounds__(256) void kgroups_last_round_kernel(const float* __restrict__ ws, int slices, int t0, int tiles_n, int tiles_m, int64_t M, int64_t N,
                                                                 float* __restrict__ Y) {
    const int j = blockIdx.x >> 3, r = 16 * (blockIdx.x & 7) + (threadIdx.x >> 4);
    int bn, bm;
    tile_of(t0 + j, tiles_n, tiles_m, bn, bm);
    const int64_t m = (int64_t)bm * kKgBM + r;
    if (m >= M) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int f = (threadIdx.x & 15) * 4 + 64 * u;
        const int64_t n = (int64_t)bn * kKgBN + f;
        if (n >= N) continue;
        const float* src = ws + (int64_t)j * slices * (kKgBM * kKgBN) + r * kKgBN + f;
        f32x4 sum = *reinterpret_cast<const f32x4*>(src);
        for (int y = 1; y < slices; ++y) sum += *reinterpret_cast<const f32x4*>(src + (int64_t)y * (kKgBM * kKgBN));
        *reinterpret_cast<f32x4*>(Y + m * N + n) = sum;
    }
}

void launch_prefill4_kgroups(const Q4Prefill& a, int split, int tail, float* ws, hipStream_t stream) {
    static const hipError_t granted[] = {kg_grant(prefill4_kgroups_kernel<128, false>), kg_grant(prefill4_kgroups_kernel<128, true>),
                                         kg_grant(prefill4_kgroups_kernel<64, false>), kg_grant(prefill4_kgroups_kernel<64, true>)};
    (void)granted;
    const int tiles_n = (int)((a.N + kKgBN - 1) / kKgBN), tiles_m = (int)((a.M + kKgBM - 1) / kKgBM), nblk = tiles_n * tiles_m;
    const auto launch = [&](int t0, int cnt, int slices, int slots, float* Y) {
        const auto kernel = slices > 1 ? a.tile == 128 ? &prefill4_kgroups_kernel<128, true> : &prefill4_kgroups_kernel<64, true>
                                       : a.tile == 128 ? &prefill4_kgroups_kernel<128, false> : &prefill4_kgroups_kernel<64, false>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)((cnt + 7) / 8 * 8), (unsigned)slices), dim3(512), kKgLds, stream, a.X, a.M, a.N, a.K, a.payload, a.scales,
                           a.table, a.Tk, tiles_n, tiles_m, t0, cnt, slots, Y);
    };
    if (tail == 0) {
        launch(0, nblk, split, 0, split > 1 ? ws : a.Y);
        return;
    }
    launch(0, nblk - tail, 1, 0, a.Y);
    launch(nblk - tail, tail, split, 1, ws);
    hipLaunchKernelGGL(kgroups_last_round_kernel, dim3((unsigned)(8 * tail)), dim3(256), 0, stream, ws, split, nblk - tail, tiles_n, tiles_m, a.M, a.N, a.Y);
}

}  // namespace patch
