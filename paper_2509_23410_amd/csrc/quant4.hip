// 4-bit weight-only storage of the hybrid dense / 2:4 weight and its decode-shaped product (Section 5.2 of the paper,
// "Quantization": the pruned model is composed with 4-bit weight-only quantization; the table there counts 4 bits per
// element of a dense tile and 2 x 4 + 4 bits per group of four of a 2:4 tile).  The paper names no quantizer; this
// library's: symmetric, 15 levels, one scale per row of a tile,
//     s = bf16(max|w| / 7),   q = clamp(rint(w / s), -7, 7)   (both in fp32, correctly rounded division, ties to even),
// and the weight the product uses is bf16(q s): the exact product rounded once.  A pruned weight keeps code 0, so a
// 2:4 tile stays 2:4; its kept positions are those of the unquantized matrix.
//
// Layout (tiles row-major, each on a 256-byte granule, table entry = offset / 256 << 1 | is 2:4, as for bf16):
//   dense tile : code fragments in (strip, K-step) order, 512 B each: lane l holds two dwords, the 8 codes of
//                W[row0 + l % 16][k0 + 8 (l / 16) + e] and those 32 columns further (the two operands of
//                v_mfma_f32_16x16x32_bf16), code e in bits [4e+3 : 4e], two's complement
//   2:4 tile   : code fragments of 256 B: lane l holds the 8 kept codes of W[row0 + l % 16][k0 + 16 (l / 16) .. + 15]
//                (the operand of v_smfmac_f32_16x16x64_bf16); then the positions, uint16 [strip][lane][K-step] as in the
//                bf16 layout
//   scales     : an array of their own, bf16 [strip of 16 rows][tile column][row in strip]: the scales a strip needs
//                along K are contiguous and no cache line is shared between strips (strips of one tile run in
//                workgroups on different XCDs; inside the tile every line of scales was fetched by four L2s)
// The product kernel dequantizes in registers (8 codes -> 8 bf16 with integer rounding) and then runs the same matrix
// instructions as the bf16 decode kernel: a workgroup owns one to three strips of 16 features, its wavefronts split K,
// partial sums meet in LDS in wavefront order (bit-reproducible); several weights sharing X run as one launch
// (patch_gemm4_many).  That kernel takes up to 64 rows of X (one, two or four blocks of 16) per pass over the weight;
// for more rows there are prefill-shaped kernels that keep the weight in 4 bits (prefill4_kernel below, prefill4_kgroups_kernel in
// quant4_kgroups.hip; patch_gemm4_ex), and any weight can be dequantized once and packed as bf16 (patch_pack_from4).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <new>
#include <vector>

#include "../../include/patch.h"
#include "batch_parts.h"
#include "epilogue.h"
#include "host_word.h"
#include "kernels.h"
#include "layout.h"
#include "map_args.h"
#include "prefill_parts.h"
#include "quant4_layout.h"
#include "saved.h"

namespace patch {

typedef __bf16 q4_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 q4_bf16x16 __attribute__((ext_vector_type(16)));
typedef float q4_f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int q4_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int q4_u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int q4_pair_t __attribute__((ext_vector_type(2), aligned(4)));   // two at a dword's
union Q4A { q4_u32x4 raw; q4_bf16x8 v; };
union Q4B { q4_u32x4 raw[2]; q4_bf16x8 h[2]; q4_bf16x16 v; };

__device__ __forceinline__ float q4_bf16_to_float(uint32_t bits) { return __uint_as_float(bits << 16); }

// 4-bit code of w for scale s (s > 0), as a nibble: rint(w / s) clamped, the quotient correctly rounded.  Where s is well
// inside the exponent range, w inv refined once rounds to the same integer as the division (about a dozen instructions):
// w and s are bf16 (8-bit significands), so their quotient is a half-integer exactly - which the refinement then
// reproduces, its residual being exact - or at least 2^-10 away from one.  inv = 1 / s to a few units in the last place.
// The quotient is at most 7 (1 + 2^-8) (s = max |w| / 7 rounded to bf16), so it needs no clamp there, and adding 1.5 x 2^23
// rounds it to an integer, ties to even, whose low bits are the sum's.
__device__ __forceinline__ uint32_t q4_code(uint16_t w_bits, float s, float inv, bool plain) {
    const float w = q4_bf16_to_float(w_bits);
    if (plain) {
        const float q0 = w * inv;
        return __float_as_uint(__builtin_fmaf(__builtin_fmaf(-q0, s, w), inv, q0) + 0x1.8p23f) & 0xFu;
    }
    return (uint32_t)((int)fminf(fmaxf(rintf(__fdiv_rn(w, s)), -7.0f), 7.0f)) & 0xFu;
}

// 8 codes of a dword -> 8 bf16 values bf16(q s), element e from bits [4e+3 : 4e].  v_cvt_off_f32_i4 turns the low nibble
// of a byte (selected by SDWA; the odd nibbles come from the dword shifted by 4) into the float q / 16 in one
// instruction - a bit-field extract and an integer conversion otherwise; q / 16 times 16 s is q s, exact in fp32
// (4 x 8 bits), and the conversion of a float pair to bf16 rounds to nearest, ties to even (v_cvt_pk_bf16_f32).
typedef __bf16 q4_bf16x2 __attribute__((ext_vector_type(2)));
typedef float q4_f32x2 __attribute__((ext_vector_type(2)));
#define PATCH_Q4_NIBBLE(dst, src, byte) \
    asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #byte : "=v"(dst) : "v"(src))
__device__ __forceinline__ q4_u32x4 q4_dequant8(uint32_t codes, float s) {
    const float s16 = s * 16.0f;
    const uint32_t odd = codes >> 4;
    float lo[4], hi[4];
    PATCH_Q4_NIBBLE(lo[0], codes, 0); PATCH_Q4_NIBBLE(lo[1], codes, 1); PATCH_Q4_NIBBLE(lo[2], codes, 2); PATCH_Q4_NIBBLE(lo[3], codes, 3);
    PATCH_Q4_NIBBLE(hi[0], odd, 0); PATCH_Q4_NIBBLE(hi[1], odd, 1); PATCH_Q4_NIBBLE(hi[2], odd, 2); PATCH_Q4_NIBBLE(hi[3], odd, 3);
    q4_u32x4 out;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const q4_f32x2 f = {lo[p] * s16, hi[p] * s16};
        const q4_bf16x2 r = __builtin_convertvector(f, q4_bf16x2);
        out[p] = *reinterpret_cast<const uint32_t*>(&r);
    }
    return out;
}
#undef PATCH_Q4_NIBBLE

__device__ __forceinline__ bool q4_nonzero(uint16_t h) { return (h & 0x7FFFu) != 0; }

// One workgroup per tile: scales and codes (and, for a 2:4 tile, the kept positions of the unquantized weights).  Bound by
// memory (2 bytes read, 0.4 - 0.5 written per weight): a thread holds its 16-byte pieces of the tile in registers, so W is read
// once, in whole rows (consecutive lanes take consecutive pieces of a row); the lanes of a row find its maximum among
// themselves; the codes are put together in LDS and leave as one contiguous run.  A first version (one thread per row for the
// maximum, the tile read again in fragment order, a division per weight) took 76 us on 11008 x 4096, tile 128, f = 0.5, and 31 us on
// 4096 x 4096, tile 64; this one 41 and 17 us (about half of that is arithmetic: eight instructions per code).
template <int TILE>
__global__ __launch_bounds__(256) void pack4_kernel(const TileMapArgs map, int first, const uint16_t* __restrict__ W, int64_t K, int Tk,
                                                    uint8_t* __restrict__ payload, uint32_t* __restrict__ table, uint16_t* __restrict__ scales,
                                                    uint32_t* __restrict__ not_24) {
    constexpr int KPT = TILE / kStepCols, SPT = TILE / kStripRows;
    constexpr int CPR = TILE / 8, RPP = 256 / CPR, PASSES = TILE / RPP;   // pieces per row, rows per pass, passes
    __shared__ __attribute__((aligned(16))) uint8_t stage[q4_dense_tile(TILE)];
    const int t = first + blockIdx.x;
    const int tn = t / Tk, tk = t % Tk;
    const uint32_t e = map_entry(map, blockIdx.x, t, q4_dense_tile(TILE), q4_sparse_tile(TILE));
    if (threadIdx.x == 0) table[t] = e;
    const bool sparse = entry_sparse(e);
    const int kc = threadIdx.x % CPR, r0 = threadIdx.x / CPR;   // piece of the row, first row
    const int j = kc >> 3;                                      // K-step of the piece
    union Piece { q4_u32x4 v; uint16_t h[8]; } in[PASSES];
    const uint16_t* src = W + ((int64_t)tn * TILE + r0) * K + (int64_t)tk * TILE + 8 * kc;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) in[p].v = *reinterpret_cast<const q4_u32x4*>(src + (int64_t)p * RPP * K);
    bool ok = true;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int row = r0 + p * RPP, strip = row >> 4, i = row & 15;
        uint32_t amax = 0;   // |w| compares like its bit pattern
#pragma unroll
        for (int k = 0; k < 8; ++k) { const uint32_t a = in[p].h[k] & 0x7FFFu; amax = a > amax ? a : amax; }
#pragma unroll
        for (int x = 1; x < CPR; x <<= 1) { const uint32_t a = __shfl_xor(amax, x); amax = a > amax ? a : amax; }
        const uint32_t sb = bf16_rne_bits(__fdiv_rn(q4_bf16_to_float(amax), 7.0f));
        if (kc == 0) scales[q4_scale_index((int64_t)tn * SPT + strip, Tk, tk, i)] = (uint16_t)sb;
        const float scl = q4_bf16_to_float(sb), inv = __builtin_amdgcn_rcpf(scl);
        const bool some = scl > 0.f, plain = scl >= 0x1p-100f && scl <= 0x1p100f;
        if (!sparse) {
            // operand h of the fragment, k = 8 q + element: one dword of eight codes
            const int h = (kc >> 2) & 1, q = kc & 3;
            uint32_t codes = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) codes |= (some ? q4_code(in[p].h[k], scl, inv, plain) : 0u) << (4 * k);
            *reinterpret_cast<uint32_t*>(stage + (strip * KPT + j) * 512 + (16 * q + i) * 8 + 4 * h) = codes;
        } else {
            // half of the 16 columns of a fragment's lane: two groups of four -> four kept codes, eight position bits
            const int lane = 16 * ((kc & 7) >> 1) + i, half = kc & 1;
            uint32_t codes = 0, idx = 0;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                // kept positions: the nonzeros, padded with the lowest-index zeros (the rule of the bf16 packer)
                bool keep[4];
                int nnz = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) { keep[c] = q4_nonzero(in[p].h[4 * g + c]); nnz += keep[c] ? 1 : 0; }
                if (nnz > 2) ok = false;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (!keep[c] && nnz < 2) { keep[c] = true; ++nnz; }
                int p0 = 0, p1 = 1;   // first and second kept position (the others exist when ok)
                uint16_t w0 = in[p].h[4 * g], w1 = in[p].h[4 * g + 1];
                int seen = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (keep[c]) {
                        if (seen == 0) { p0 = c; w0 = in[p].h[4 * g + c]; }
                        else if (seen == 1) { p1 = c; w1 = in[p].h[4 * g + c]; }
                        ++seen;
                    }
                const uint32_t c0 = some ? q4_code(w0, scl, inv, plain) : 0u, c1 = some ? q4_code(w1, scl, inv, plain) : 0u;
                codes |= (c0 | (c1 << 4)) << (8 * g);
                idx |= (uint32_t)(p0 | (p1 << 2)) << (4 * g);
            }
            *reinterpret_cast<uint16_t*>(stage + (strip * KPT + j) * 256 + lane * 4 + 2 * half) = (uint16_t)codes;
            stage[q4_sparse_codes(TILE) + ((strip * 64 + lane) * KPT + j) * 2 + half] = (uint8_t)idx;
        }
    }
    if (!ok) report_not_24(not_24);
    __syncthreads();
    q4_u32x4* out = reinterpret_cast<q4_u32x4*>(payload + entry_offset(e));
    const int n16 = (sparse ? q4_sparse_tile(TILE) : q4_dense_tile(TILE)) / 16;
    for (int c = threadIdx.x; c < n16; c += 256) out[c] = reinterpret_cast<const q4_u32x4*>(stage)[c];
}

// The inverse: the dequantized bf16 matrix and / or the codes (int8, 0 at dropped positions) and scales in matrix order.  Bound
// by memory, mostly by what it writes: the tile's codes pass through LDS, then a thread turns eight consecutive columns of a row
// into one 16-byte and one 8-byte store, consecutive lanes side by side (4096 x 4096, tile 64, all three outputs: 14 us, 4.2 TB/s; with
// 2-byte and 1-byte stores 62 us; 11008 x 4096, tile 128: 30 us against 161).  `codes_out` has no alignment of its own: where it is not 8-byte aligned its bytes go one by one.
template <int TILE>
__global__ __launch_bounds__(256) void unpack4_kernel(const uint8_t* __restrict__ payload, const uint16_t* __restrict__ scales,
                                                      const uint32_t* __restrict__ table, int Tk, int64_t K, uint16_t* __restrict__ W_deq,
                                                      int8_t* __restrict__ codes_out, uint16_t* __restrict__ scales_out) {
    constexpr int KPT = TILE / kStepCols, SPT = TILE / kStripRows;
    constexpr int CPR = TILE / 8, RPP = 256 / CPR, PASSES = TILE / RPP;
    __shared__ __attribute__((aligned(16))) uint8_t stage[q4_dense_tile(TILE)];
    const int t = blockIdx.x;
    const int tn = t / Tk, tk = t % Tk;
    const uint32_t e = table[t];
    const bool sparse = entry_sparse(e);
    const q4_u32x4* src = reinterpret_cast<const q4_u32x4*>(payload + entry_offset(e));
    const int n16 = (sparse ? q4_sparse_tile(TILE) : q4_dense_tile(TILE)) / 16;
    for (int c = threadIdx.x; c < n16; c += 256) reinterpret_cast<q4_u32x4*>(stage)[c] = src[c];
    // the tile columns of a tile row share the rows of the scale matrix among them: whole rows, contiguous stores
    if (scales_out)
        for (int r = tk; r < TILE; r += Tk)
            for (int c = threadIdx.x; c < Tk; c += 256)
                scales_out[((int64_t)tn * TILE + r) * Tk + c] = scales[q4_scale_index((int64_t)tn * SPT + (r >> 4), Tk, c, r & 15)];
    __syncthreads();
    const int kc = threadIdx.x % CPR, r0 = threadIdx.x / CPR, j = kc >> 3;
    const bool bytewise = (reinterpret_cast<uintptr_t>(codes_out) & 7u) != 0;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int row = r0 + p * RPP, strip = row >> 4, i = row & 15;
        const float scl = q4_bf16_to_float(scales[q4_scale_index((int64_t)tn * SPT + strip, Tk, tk, i)]);
        int qv[8];
        if (!sparse) {
            const int h = (kc >> 2) & 1, q = kc & 3;
            const uint32_t d = *reinterpret_cast<const uint32_t*>(stage + (strip * KPT + j) * 512 + (16 * q + i) * 8 + 4 * h);
#pragma unroll
            for (int k = 0; k < 8; ++k) qv[k] = ((int)(d << (28 - 4 * k))) >> 28;
        } else {
            const int lane = 16 * ((kc & 7) >> 1) + i, half = kc & 1;
            const uint32_t d = *reinterpret_cast<const uint16_t*>(stage + (strip * KPT + j) * 256 + lane * 4 + 2 * half);
            const uint32_t idx = stage[q4_sparse_codes(TILE) + ((strip * 64 + lane) * KPT + j) * 2 + half];
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int p0 = (idx >> (4 * g)) & 3, p1 = (idx >> (4 * g + 2)) & 3;
                const int c0 = ((int)(d << (28 - 8 * g))) >> 28, c1 = ((int)(d << (24 - 8 * g))) >> 28;
#pragma unroll
                for (int c = 0; c < 4; ++c) qv[4 * g + c] = c == p1 ? c1 : c == p0 ? c0 : 0;
            }
        }
        const int64_t at = ((int64_t)tn * TILE + row) * K + (int64_t)tk * TILE + 8 * kc;
        if (W_deq) {
            q4_u32x4 w;
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = bf16_pair((float)qv[2 * k] * scl, (float)qv[2 * k + 1] * scl);
            *reinterpret_cast<q4_u32x4*>(W_deq + at) = w;
        }
        if (codes_out) {
            if (bytewise) {
#pragma unroll
                for (int k = 0; k < 8; ++k) codes_out[at + k] = (int8_t)qv[k];
            } else {
                q4_u32x2 b = {0u, 0u};
#pragma unroll
                for (int k = 0; k < 8; ++k) b[k >> 2] |= ((uint32_t)qv[k] & 0xFFu) << (8 * (k & 3));
                *reinterpret_cast<q4_u32x2*>(codes_out + at) = b;
            }
        }
    }
}

// Up to 16 RB rows of X (RB = 1 .. 4 blocks of 16 rows) against the 4-bit weight in one pass over it.  A workgroup
// owns R consecutive strips of 16 features (the registers hold R x RB accumulators and RB X operands per step: R <= 3,
// with two row blocks R <= 4); its KW wavefronts take contiguous runs of 64-column steps.  A wavefront loads
// the X operand of a step once and uses it for all R strips (at 4 bits per weight X is the larger stream, so this
// reuse is what bounds the traffic), works in batches of NB steps (2; 1 when R RB > 1) and issues the next batch's loads before it
// consumes the current one.  Two batch buffers alternate; no copies.
constexpr int kQ4MaxR = 3;
constexpr int kQ4Rows = 64;   // rows of X per launch at most

template <int R, int RB, int NB>
struct Q4Batch {
    uint32_t e[NB][R];
    q4_pair_t d[NB][R];        // codes (the second dword: q4_loads with ARMS, dense)
    uint32_t p[NB][R];         // 2:4: positions; dense without ARMS: the second dword of codes
    uint32_t sc[NB][R];        // scale bits
    q4_u32x4 x[NB][RB][2];
};

// The product kernel's pointers carry their address space: the weight pointers reach it inside a by-value struct and
// pass through scalar selects, after which the compiler no longer knows that they are global (it then emits flat
// loads) nor that the table is not written by the kernel (it then reads entries with vector loads).  Table entries
// are read through the constant address space (scalar loads), everything else through the global one.
#define PATCH_Q4_GLOBAL __attribute__((address_space(1)))
#define PATCH_Q4_CONST __attribute__((address_space(4)))
typedef const PATCH_Q4_CONST uint32_t* q4_table_ptr;
typedef const PATCH_Q4_GLOBAL uint8_t* q4_bytes_ptr;
typedef const PATCH_Q4_GLOBAL uint16_t* q4_u16_ptr;

template <int R>
struct Q4Strips {
    q4_table_ptr row[R];      // table entries of the strip's tile row
    q4_bytes_ptr pay[R];      // payload of the strip's weight
    int s[R];                 // strip within the tile
    q4_u16_ptr scl[R];        // this lane's scale of the strip for tile column 0 (the next column is 16 scales on)
};

// Steps past the wavefront's run repeat its last step (in bounds; discarded by q4_compute).
template <int TILE, int R, int NB>
__device__ __forceinline__ void q4_entries(uint32_t (&e)[NB][R], const Q4Strips<R>& st, int step0, int last) {
    constexpr int KPT = TILE / kStepCols;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int step = step0 + i < last ? step0 + i : last;
#pragma unroll
        for (int r = 0; r < R; ++r) e[i][r] = st.row[r][step / KPT];
    }
}

// The loads of a batch whose entries q4_entries has filled in.  Either no load is conditional, a dense lane's two dwords one load each, or (ARMS) a
// dense lane's come by one load behind a branch.  Both arms then issue two loads: the compiler knows how many are in flight only if they are as many,
// and would otherwise wait for all of them.  The branches cost a wavefront more issue time than the wider load saves unless it runs for a while
// (27 x 2 x 3 single weights, 11 row counts, ARMS against none, mean ratio at f = 0 / 1/2 / 1: 2 steps a wavefront 1.025 / 1.027 / 1.028, 4 steps
// 0.99 / 1.00 / 1.01, 5 and more 0.967 / 0.981 / 1.001; f = 0, 9 rows, mask tile 64: 512 x 13824 13.7 -> 12.9 us).
template <int TILE, int R, int RB, int NB, bool ARMS>
__device__ __forceinline__ void q4_loads(Q4Batch<R, RB, NB>& b, const Q4Strips<R>& st, const q4_u16_ptr (&xrow)[RB], int lane, int step0, int last) {
    constexpr int KPT = TILE / kStepCols;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int step = step0 + i < last ? step0 + i : last;
        const int j = step % KPT;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            b.x[i][rb][0] = *reinterpret_cast<const PATCH_Q4_GLOBAL q4_u32x4*>(xrow[rb] + (int64_t)step * kStepCols);
            b.x[i][rb][1] = *reinterpret_cast<const PATCH_Q4_GLOBAL q4_u32x4*>(xrow[rb] + (int64_t)step * kStepCols + 32);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            q4_bytes_ptr base = st.pay[r] + entry_offset(b.e[i][r]);
            const int s = st.s[r];
            b.sc[i][r] = st.scl[r][(step / KPT) * 16];
            // positions on mask tile 64: a dword is shared with the neighbour
            const bool sp = entry_sparse(b.e[i][r]);
            const int f = s * KPT + j;
            if constexpr (ARMS) {
                if (sp) {
                    b.d[i][r][0] = *reinterpret_cast<const PATCH_Q4_GLOBAL uint32_t*>(base + f * 256 + lane * 4);
                    b.p[i][r] = *reinterpret_cast<const PATCH_Q4_GLOBAL uint32_t*>(base + q4_sparse_codes(TILE) + (TILE == 128 ? (s * 64 + lane) * 4 : (s * 32 + (lane >> 1)) * 4));
                } else {
                    b.d[i][r] = *reinterpret_cast<const PATCH_Q4_GLOBAL q4_pair_t*>(base + f * 512 + lane * 8);
                    b.p[i][r] = *reinterpret_cast<const PATCH_Q4_GLOBAL uint32_t*>(base);   // not used
                }
            } else {
                b.d[i][r][0] = *reinterpret_cast<const PATCH_Q4_GLOBAL uint32_t*>(base + (sp ? f * 256 + lane * 4 : f * 512 + lane * 8));
                b.p[i][r] = *reinterpret_cast<const PATCH_Q4_GLOBAL uint32_t*>(
                    base + (sp ? q4_sparse_codes(TILE) + (TILE == 128 ? (s * 64 + lane) * 4 : (s * 32 + (lane >> 1)) * 4) : f * 512 + lane * 8 + 4));
            }
        }
    }
}

template <int TILE, int R, int RB, int NB, bool ARMS>
__device__ __forceinline__ void q4_compute(const Q4Batch<R, RB, NB>& b, q4_f32x4 (&acc)[R][RB], int lane, int step0, int end) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (step0 + i >= end) break;   // uniform
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float scl = q4_bf16_to_float(b.sc[i][r]);
            if (!entry_sparse(b.e[i][r])) {
                Q4A a0, a1;
                a0.raw = q4_dequant8(b.d[i][r][0], scl);
                a1.raw = q4_dequant8(ARMS ? b.d[i][r][1] : b.p[i][r], scl);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    Q4B x;
                    x.raw[0] = b.x[i][rb][0];
                    x.raw[1] = b.x[i][rb][1];
                    acc[r][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0.v, x.h[0], acc[r][rb], 0, 0, 0);
                    acc[r][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1.v, x.h[1], acc[r][rb], 0, 0, 0);
                }
            } else {
                Q4A a;
                a.raw = q4_dequant8(b.d[i][r][0], scl);
                const int pos = (int)(b.p[i][r] >> (16 * (TILE == 128 ? (step0 + i) & 1 : lane & 1)));
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    Q4B x;
                    x.raw[0] = b.x[i][rb][0];
                    x.raw[1] = b.x[i][rb][1];
                    acc[r][rb] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a.v, x.v, acc[r][rb], pos, 0, 0);
                }
            }
        }
    }
}

// Up to MAXC 4-bit weights that share one X (same K, same tile) in one launch.  The launch numbers the 16-feature strips
// across all weights (first[i] = first strip of weight i, total = their number); a workgroup takes R consecutive
// strips, which may belong to two weights.
template <int MAXC>
struct Q4Set {
    static constexpr int kMax = MAXC;
    const uint8_t* payload[MAXC];
    const uint16_t* scales[MAXC];
    const uint32_t* table[MAXC];
    float* Y[MAXC];
    int64_t N[MAXC];
    int first[MAXC];
    int count, total;
};

// A set of one: 40 bytes of kernel arguments.
struct Q4One {
    const uint8_t* payload;
    const uint16_t* scales;
    const uint32_t* table;
    float* Y;
    int64_t N;
};

struct Q4Weight {
    uint64_t payload, scales, table, Y;
    int64_t N;
    int first;
};

// The weight that strip g of the launch belongs to (g uniform): scalar selects over the candidates, so that every
// pointer stays in scalar registers.
template <typename SetT>
__device__ __forceinline__ Q4Weight q4_weight_of(const SetT& set, int g) {
    Q4Weight wt;
    if constexpr (sizeof(SetT) == sizeof(Q4One)) {
        wt = Q4Weight{reinterpret_cast<uint64_t>(set.payload), reinterpret_cast<uint64_t>(set.scales), reinterpret_cast<uint64_t>(set.table),
                      reinterpret_cast<uint64_t>(set.Y), set.N, 0};
    } else {
        wt = Q4Weight{reinterpret_cast<uint64_t>(set.payload[0]), reinterpret_cast<uint64_t>(set.scales[0]),
                      reinterpret_cast<uint64_t>(set.table[0]), reinterpret_cast<uint64_t>(set.Y[0]), set.N[0], 0};
#pragma unroll
        for (int i = 1; i < SetT::kMax; ++i) {
            const bool here = i < set.count && g >= set.first[i];
            wt.payload = here ? reinterpret_cast<uint64_t>(set.payload[i]) : wt.payload;
            wt.scales = here ? reinterpret_cast<uint64_t>(set.scales[i]) : wt.scales;
            wt.table = here ? reinterpret_cast<uint64_t>(set.table[i]) : wt.table;
            wt.Y = here ? reinterpret_cast<uint64_t>(set.Y[i]) : wt.Y;
            wt.N = here ? set.N[i] : wt.N;
            wt.first = here ? set.first[i] : wt.first;
        }
    }
    return wt;
}

// Every kernel argument is requested in the kernel's first instructions and waited for once (the compiler otherwise
// fetches an argument where it is first used, e.g. behind a branch: one more, if short, round trip before the first
// weight load).  What costs far more is losing the address spaces (see PATCH_Q4_GLOBAL above): with flat loads and
// table entries read by vector loads the same launch took 8.0 us instead of 6.2.
#define PATCH_Q4_ARGS_NOW(...) asm volatile("" ::__VA_ARGS__)

// wavefronts per workgroup at most: 16, or 8 with four or more accumulators and X operands of several row blocks
// (whose registers do not fit 16 times into a compute unit)
constexpr int q4_max_waves(int R, int RB) { return RB == 4 || R * RB > 4 || (RB == 2 && R > 1) ? 8 : 16; }

template <int TILE, int R, int RB, typename SetT, bool ARMS>
__global__ __launch_bounds__(64 * q4_max_waves(R, RB)) void decode4_kernel(const uint16_t* __restrict__ X, int64_t m0, int rows, int64_t K, int Tk, int KW,
                                                       const SetT set) {
    constexpr bool kOne = sizeof(SetT) == sizeof(Q4One);
    constexpr int KPT = TILE / kStepCols, SPT = TILE / kStripRows;
    constexpr int NB = RB > 1 || R > 1 ? 1 : 2;   // steps per batch
    constexpr int CH = R * RB < 8 ? R * RB : 8;   // items per round of the final reduction
    __shared__ q4_f32x4 red[CH][q4_max_waves(R, RB)][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // of KW wavefronts: an argument (the launch size is a hidden one, fetched apart)
    const int col = lane & 15, q = lane >> 4;
    int total_strips;
    if constexpr (kOne) total_strips = (int)(set.N / kStripRows);
    else total_strips = set.total;
    const int g0 = (int)blockIdx.x * R;
    Q4Strips<R> st;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int g = g0 + r < total_strips ? g0 + r : total_strips - 1;   // a strip past the end repeats the last one (not stored)
        const Q4Weight wt = q4_weight_of(set, g);
        PATCH_Q4_ARGS_NOW("s"(wt.payload), "s"(wt.scales), "s"(wt.table), "s"(wt.first));
        const int strip = g - wt.first;
        st.row[r] = reinterpret_cast<q4_table_ptr>(wt.table) + (int64_t)(strip / SPT) * Tk;
        st.pay[r] = reinterpret_cast<q4_bytes_ptr>(wt.payload);
        st.s[r] = strip % SPT;
        st.scl[r] = reinterpret_cast<q4_u16_ptr>(wt.scales) + q4_scale_index(strip, Tk, 0, col);
    }
    // the first (strip, row block) this wavefront adds up and stores at the end (it takes items w, w + KW, ...)
    {
        const int gw = g0 + (w < R * RB ? w / RB : 0);
        const Q4Weight wy = q4_weight_of(set, gw < total_strips ? gw : total_strips - 1);
        PATCH_Q4_ARGS_NOW("s"(X), "s"(m0), "s"(rows), "s"(K), "s"(Tk), "s"(KW), "s"(wy.Y), "s"(wy.N), "s"(wy.first));
    }
    const int total = Tk * KPT, per = (total + KW - 1) / KW;
    const int begin = w * per, end = begin + per < total ? begin + per : total;
    q4_u16_ptr xrow[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int m = 16 * rb + col < rows ? 16 * rb + col : rows - 1;   // columns without a row: any valid row, not stored
        xrow[rb] = reinterpret_cast<q4_u16_ptr>(reinterpret_cast<uintptr_t>(X)) + (m0 + m) * K + 8 * q;
    }
    q4_f32x4 acc[R][RB];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[r][rb] = q4_f32x4{0.f, 0.f, 0.f, 0.f};
    if (begin < end) {
        // Two batches alternate, one requested before the one in front of it is multiplied, table entries two batches further ahead.  No load is
        // conditional - behind a branch the compiler waits for the loads of either arm, i.e. for the batch just requested - so the last one or
        // two batches are written out.  (With conditional loads, f = 1/2: two 13824 x 5120 at 24 rows 39.4 -> 33.6 us here, three 896 x 896 at 16 / 40
        // rows 3.9 / 5.7 -> 3.4 / 4.8, 4096 x 11008 at 16 rows 17.1 -> 16.0.)
        Q4Batch<R, RB, NB> b0, b1;
        uint32_t e2[NB][R], e3[NB][R];
        auto take = [&](uint32_t (&to)[NB][R], const uint32_t (&from)[NB][R]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int r = 0; r < R; ++r) to[i][r] = from[i][r];
        };
        q4_entries<TILE, R, NB>(b0.e, st, begin, end - 1);
        q4_entries<TILE, R, NB>(b1.e, st, begin + NB, end - 1);
        q4_entries<TILE, R, NB>(e2, st, begin + 2 * NB, end - 1);
        q4_entries<TILE, R, NB>(e3, st, begin + 3 * NB, end - 1);
        q4_loads<TILE, R, RB, NB, ARMS>(b0, st, xrow, lane, begin, end - 1);
        int step0 = begin;
        auto two_batches = [&]() __attribute__((always_inline)) {
            q4_loads<TILE, R, RB, NB, ARMS>(b1, st, xrow, lane, step0 + NB, end - 1);
            q4_compute<TILE, R, RB, NB, ARMS>(b0, acc, lane, step0, end);
            take(b0.e, e2);
            q4_entries<TILE, R, NB>(e2, st, step0 + 4 * NB, end - 1);
            q4_loads<TILE, R, RB, NB, ARMS>(b0, st, xrow, lane, step0 + 2 * NB, end - 1);
            q4_compute<TILE, R, RB, NB, ARMS>(b1, acc, lane, step0 + NB, end);
            take(b1.e, e3);
            q4_entries<TILE, R, NB>(e3, st, step0 + 5 * NB, end - 1);
        };
        // With the test at the top the compiler copies the batch just requested at every turn - waits for it and holds it twice - in some kernels for
        // mask tile 128 (R = 3, RB = 4 in a set of more than three: 256 vector registers and 236 bytes of scratch per lane, 194 as do .. while; R = 3,
        // RB = 1 in a set 119, 78).  f = 1/2: four 2560 x 2560 at 16 / 32 / 64 rows 9.9 / 11.9 / 36.4 -> 9.4 / 10.9 / 16.9 us, 4864 / 4864 / 896 / 896 x 896 at
        // 64 17.2 -> 9.2, three 896 x 896 at 16 4.0 -> 3.7.  On mask tile 64 it never did: there do .. while saves registers from R RB = 6 on
        // (R = 3, RB = 2: 127, 115) and is 0.5 % slower below (10 % of the calls 2 - 7 %).
        if constexpr (TILE == 128 || R * RB > 4) {
            if (step0 + 2 * NB < end) do {
                two_batches();
                step0 += 2 * NB;
            } while (step0 + 2 * NB < end);
        } else {
            for (; step0 + 2 * NB < end; step0 += 2 * NB) two_batches();
        }
        if (step0 + NB < end) {
            q4_loads<TILE, R, RB, NB, ARMS>(b1, st, xrow, lane, step0 + NB, end - 1);
            q4_compute<TILE, R, RB, NB, ARMS>(b0, acc, lane, step0, end);
            q4_compute<TILE, R, RB, NB, ARMS>(b1, acc, lane, step0 + NB, end);
        } else {
            q4_compute<TILE, R, RB, NB, ARMS>(b0, acc, lane, step0, end);
        }
    }
    // Partial sums meet in LDS, CH (strip, row block) items at a time (all of them unless R RB > 8): wavefront w adds
    // up the items w, w + KW, ... of the chunk in wavefront order and stores them.
#pragma unroll
    for (int c0 = 0; c0 < R * RB; c0 += CH) {
        if (c0 > 0) __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                if (r * RB + rb >= c0 && r * RB + rb < c0 + CH) red[r * RB + rb - c0][w][lane] = acc[r][rb];
        __syncthreads();
        for (int i0 = w; i0 < CH && c0 + i0 < R * RB; i0 += KW) {
            const int item = c0 + i0, gw = g0 + item / RB, wrb = item % RB;
            if (gw >= total_strips) break;
            const Q4Weight wy = q4_weight_of(set, gw);
            const q4_f32x4 sum = sum_in_order(KW, [&](int i) { return red[i0][i][lane]; });
            PATCH_Q4_GLOBAL float* Yg = reinterpret_cast<PATCH_Q4_GLOBAL float*>(wy.Y);
            if (16 * wrb + col < rows)
                *reinterpret_cast<PATCH_Q4_GLOBAL q4_f32x4*>(Yg + (m0 + 16 * wrb + col) * wy.N + (int64_t)(gw - wy.first) * 16 + 4 * q) = sum;
        }
    }
}

template <int TILE, int R, int RB, typename SetT>
static void launch_decode4(const uint16_t* X, int64_t m0, int rows, int64_t K, int Tk, const SetT& set, int groups, int kw, hipStream_t s) {
    // the wider loads of dense tiles: a single weight and more than four steps per wavefront (q4_loads)
    constexpr bool kOne = sizeof(SetT) == sizeof(Q4One);
    auto* kernel = kOne && Tk * (TILE / kStepCols) > 4 * kw ? decode4_kernel<TILE, R, RB, SetT, kOne> : decode4_kernel<TILE, R, RB, SetT, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3((unsigned)(kw * 64)), 0, s, X, m0, rows, K, Tk, kw, set);
}

// up to 3 strips per workgroup, up to 4 with two blocks of 16 rows
template <int TILE, typename SetT>
static void launch_decode4_r(int R, int RB, const uint16_t* X, int64_t m0, int rows, int64_t K, int Tk, const SetT& set, int groups, int kw,
                             hipStream_t s) {
#define PATCH_Q4_CASE(r, rb) \
    if (R == r && RB == rb) return launch_decode4<TILE, r, rb, SetT>(X, m0, rows, K, Tk, set, groups, kw, s)
    PATCH_Q4_CASE(1, 1); PATCH_Q4_CASE(2, 1); PATCH_Q4_CASE(3, 1);
    PATCH_Q4_CASE(1, 2); PATCH_Q4_CASE(2, 2); PATCH_Q4_CASE(3, 2); PATCH_Q4_CASE(4, 2);
    PATCH_Q4_CASE(1, 3); PATCH_Q4_CASE(2, 3); PATCH_Q4_CASE(3, 3);
    PATCH_Q4_CASE(1, 4); PATCH_Q4_CASE(2, 4); PATCH_Q4_CASE(3, 4);
#undef PATCH_Q4_CASE
}

// ---- the same for mask tile 128 and up to 8 rows, a whole tile (128 columns) of a strip at a time
//
// What bounds a launch of so few rows is requests and their latency, not bytes: per 64-column step the kernel above issues a load of codes,
// one of scales, one of positions and two of X.  Here a lane takes what lies side by side in the strip's stored codes - its 16 (2:4: 8)
// bytes hold rows 2 a and 2 a + 1 of one K-step, a = lane % 8 - so that a tile is two loads of codes (2:4: codes, positions) and one of
// scales.  The matrix instructions then see
//     A (weights), lane 16 g + r:  row 2 (r % 8) + c of the strip, K-step r / 8, k = 8 g + e (+ 32: second operand; 2:4: 16 g ..)
//     B (X), lane 16 g + n:        row n / 2 of X, K-step n % 2
//     D, row r, column n:          a partial sum of output (2 (r % 8) + c, n / 2) where n % 2 = r / 8 (the other half is not used)
// once for c = 0 and once for c = 1: as many instructions as before, with the 16 columns holding two K-steps of 8 rows instead of one of 16.
// With at most 4 rows the other 8 columns hold the X of the next tile, turned into place before use (a DPP move per register).
// f = 1/2, one row, decode4_kernel with conditional loads -> this kernel, us: three 4096 x 4096 11.8 -> 8.7, 4096 x 4096 5.3 -> 4.9, two
// 11008 x 4096 18.9 -> 13.5, 4096 x 11008 11.5 -> 8.6, two 13824 x 5120 27.1 -> 19.8.  What is left is the conversion (2.7 vector
// instructions a weight; a build without it 1.9 us faster on two 11008 x 4096), position and scale loads (1.8 and 0.9) and X (0.7).  Four tiles
// in flight instead of two gained nothing.
template <int R>
struct Q4Tile {
    uint32_t e[R];
    q4_pair_t d0[R];          // dense: row 2 a (two operands); 2:4: kept codes of rows 2 a, 2 a + 1
    q4_pair_t d1[R];          // dense: row 2 a + 1; 2:4: positions of the two rows, both K-steps
    uint32_t sc[R];           // scales of the two rows
};

template <int R>
__device__ __forceinline__ void q4_tile_loads(Q4Tile<R>& b, const Q4Strips<R>& st, uint32_t vcode, uint32_t vpos, int t) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool sp = entry_sparse(b.e[r]);
        const q4_bytes_ptr base = st.pay[r] + entry_offset(b.e[r]) + st.s[r] * (sp ? 512 : 1024);
        b.d0[r] = __builtin_nontemporal_load(reinterpret_cast<const PATCH_Q4_GLOBAL q4_pair_t*>(base + (vcode >> (sp ? 1 : 0))));
        b.d1[r] = __builtin_nontemporal_load(reinterpret_cast<const PATCH_Q4_GLOBAL q4_pair_t*>(base + (sp ? q4_sparse_codes(128) - st.s[r] * 256 + vpos : 8 + vcode)));
        b.sc[r] = *reinterpret_cast<const PATCH_Q4_GLOBAL uint32_t*>(st.scl[r] + t * 16);
    }
}

// dst[lane] = v[lane + 8] within each row of 16 lanes
__device__ __forceinline__ q4_u32x4 q4_rows_up8(q4_u32x4 v) {
    q4_u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v[i], 0x128, 0xF, 0xF, false);   // row_ror:8
    return r;
}

template <int R>
__device__ __forceinline__ void q4_tile_compute(const Q4Tile<R>& b, const Q4B& x, q4_f32x4 (&acc)[R][2], int jshift) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float s0 = __uint_as_float(b.sc[r] << 16), s1 = __uint_as_float(b.sc[r] & 0xFFFF0000u);
        if (!entry_sparse(b.e[r])) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                Q4A a0, a1;
                a0.raw = q4_dequant8(c ? b.d1[r][0] : b.d0[r][0], c ? s1 : s0);
                a1.raw = q4_dequant8(c ? b.d1[r][1] : b.d0[r][1], c ? s1 : s0);
                acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0.v, x.h[0], acc[r][c], 0, 0, 0);
                acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1.v, x.h[1], acc[r][c], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                Q4A a;
                a.raw = q4_dequant8(b.d0[r][c], c ? s1 : s0);
                acc[r][c] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a.v, x.v, acc[r][c], (int)(b.d1[r][c] >> jshift), 0, 0);
            }
        }
    }
}

constexpr int kQ4TileWaves = 16;

// At most XR = 4 or 8 rows of X
template <int R, int XR, typename SetT>
__global__ __launch_bounds__(64 * kQ4TileWaves) void decode4_tile_kernel(const uint16_t* __restrict__ X, int64_t m0, int rows, int64_t K, int Tk, int KW, int per,
                                                                         const SetT set) {
    constexpr bool kOne = sizeof(SetT) == sizeof(Q4One);
    constexpr int SPT = 128 / kStripRows;
    constexpr int XT = XR == 4 ? 2 : 1;   // tiles per X load
    __shared__ q4_f32x4 red[R][kQ4TileWaves][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int a = lane & 7, j = (lane >> 3) & 1, g = lane >> 4, n = lane & 15;
    int total_strips;
    if constexpr (kOne) total_strips = (int)(set.N / kStripRows);
    else total_strips = set.total;
    const int g0 = (int)blockIdx.x * R;
    Q4Strips<R> st;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int gs = g0 + r < total_strips ? g0 + r : total_strips - 1;   // a strip past the end repeats the last one (not stored)
        const Q4Weight wt = q4_weight_of(set, gs);
        PATCH_Q4_ARGS_NOW("s"(wt.payload), "s"(wt.scales), "s"(wt.table), "s"(wt.first));
        const int strip = gs - wt.first;
        st.row[r] = reinterpret_cast<q4_table_ptr>(wt.table) + (int64_t)(strip / SPT) * Tk;
        st.pay[r] = reinterpret_cast<q4_bytes_ptr>(wt.payload);
        st.s[r] = strip % SPT;
        st.scl[r] = reinterpret_cast<q4_u16_ptr>(wt.scales) + q4_scale_index(strip, Tk, 0, 2 * a);
    }
    {
        const int gw = g0 + (w < R ? w : 0);
        const Q4Weight wy = q4_weight_of(set, gw < total_strips ? gw : total_strips - 1);
        PATCH_Q4_ARGS_NOW("s"(X), "s"(m0), "s"(rows), "s"(K), "s"(Tk), "s"(KW), "s"(per), "s"(wy.Y), "s"(wy.N), "s"(wy.first));
    }
    const uint32_t vcode = (uint32_t)(j * 32 + g * 8 + a) * 16, vpos = (uint32_t)(16 * g + 2 * a) * 4;
    const int begin = w * per, end = begin + per < Tk ? begin + per : Tk;   // per = ceil(Tk / KW)
    const int last = end - 1;
    // this lane's row of X and tile of a load; columns without a row: any valid row, not stored
    const int xt = XT == 2 ? n >> 3 : 0;
    const int xm = (n >> 1) % XR;
    const q4_bytes_ptr xrow = reinterpret_cast<q4_bytes_ptr>(reinterpret_cast<uintptr_t>(X)) + ((m0 + (xm < rows ? xm : rows - 1)) * K + 64 * (n & 1) + 8 * g) * 2;
    q4_f32x4 acc[R][2];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r][0] = acc[r][1] = q4_f32x4{0.f, 0.f, 0.f, 0.f};
    if (begin < end) {
        // Two buffers alternate, a tile requested before the one in front of it is multiplied; table entries two tiles further ahead.  No load
        // is conditional (behind a branch the compiler would wait for the loads of either arm, i.e. for the tile just requested), so the
        // last one or two tiles are written out.
        Q4Tile<R> b0, b1;
        uint32_t e2[R], e3[R];
        Q4B x0, x1;   // X of b0's and b1's tile, or (XT = 2) of both and of the next two
        auto entries = [&](uint32_t (&e)[R], int t) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < R; ++r) e[r] = st.row[r][t < last ? t : last];
        };
        auto load = [&](Q4Tile<R>& b, int t) __attribute__((always_inline)) { q4_tile_loads<R>(b, st, vcode, vpos, t); };
        auto load_x = [&](Q4B& x, int t) __attribute__((always_inline)) {
            if constexpr (XT == 2) t = t + xt < last ? t + xt : last;
            const int64_t off = (int64_t)t * 256;
            x.raw[0] = *reinterpret_cast<const PATCH_Q4_GLOBAL q4_u32x4*>(xrow + off);
            x.raw[1] = *reinterpret_cast<const PATCH_Q4_GLOBAL q4_u32x4*>(xrow + off + 64);
        };
        auto second = [&]() __attribute__((always_inline)) {   // b1's tile
            if constexpr (XT == 2) {
                Q4B up;
                up.raw[0] = q4_rows_up8(x0.raw[0]);
                up.raw[1] = q4_rows_up8(x0.raw[1]);
                q4_tile_compute<R>(b1, up, acc, 16 * j);
            } else {
                q4_tile_compute<R>(b1, x1, acc, 16 * j);
            }
        };
        entries(b0.e, begin);
        entries(b1.e, begin + 1);
        entries(e2, begin + 2);
        entries(e3, begin + 3);
        load_x(x0, begin);
        load(b0, begin);
        int t = begin;
        for (; t + 2 < end; t += 2) {
            if constexpr (XT == 1) load_x(x1, t + 1);
            load(b1, t + 1);
            q4_tile_compute<R>(b0, x0, acc, 16 * j);
#pragma unroll
            for (int r = 0; r < R; ++r) b0.e[r] = e2[r];
            entries(e2, t + 4);
            if constexpr (XT == 1) load_x(x0, t + 2);
            else load_x(x1, t + 2);
            load(b0, t + 2);
            second();
            if constexpr (XT == 2) x0 = x1;
#pragma unroll
            for (int r = 0; r < R; ++r) b1.e[r] = e3[r];
            entries(e3, t + 5);
        }
        if (t + 1 < end) {
            if constexpr (XT == 1) load_x(x1, t + 1);
            load(b1, t + 1);
            q4_tile_compute<R>(b0, x0, acc, 16 * j);
            second();
        } else {
            q4_tile_compute<R>(b0, x0, acc, 16 * j);
        }
    }
    // Partial sums meet in LDS, the used half of a product (columns n with n % 2 = row / 8) in 32 places per c; wavefront w adds up
    // strip w in wavefront order, then the two K-steps, and stores 4 features per lane.
    if ((n & 1) == (g >> 1) && n < 2 * XR)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c) red[r][w][32 * c + 8 * g + (n >> 1)] = acc[r][c];
    __syncthreads();
    if (const int gw = g0 + w; w < R && gw < total_strips) {
        const Q4Weight wy = q4_weight_of(set, gw);
        // lane 32 c + 16 p + 8 h + m: row m, K-step p, features 8 h + 2 i + c
        const int c = lane >> 5, h = (lane >> 3) & 1, m = lane & 7;
        q4_f32x4 sum = sum_in_order(KW, [&](int i) { return red[w][i][lane]; });
        q4_f32x4 other;
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] += __shfl_xor(sum[i], 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) other[i] = __shfl_xor(sum[i], 32);
        const q4_f32x4 out = c == 0 ? q4_f32x4{sum[0], other[0], sum[1], other[1]} : q4_f32x4{other[2], sum[2], other[3], sum[3]};
        PATCH_Q4_GLOBAL float* Yg = reinterpret_cast<PATCH_Q4_GLOBAL float*>(wy.Y);
        if (!(lane & 16) && m < rows)
            *reinterpret_cast<PATCH_Q4_GLOBAL q4_f32x4*>(Yg + (m0 + m) * wy.N + (int64_t)(gw - wy.first) * 16 + 8 * h + 4 * c) = out;
    }
}

template <int R, int XR, typename SetT>
static void launch_decode4_tile(const uint16_t* X, int64_t m0, int rows, int64_t K, int Tk, const SetT& set, int groups, int kw, hipStream_t s) {
    hipLaunchKernelGGL((decode4_tile_kernel<R, XR, SetT>), dim3((unsigned)groups), dim3((unsigned)(kw * 64)), 0, s, X, m0, rows, K, Tk, kw, (Tk + kw - 1) / kw, set);
}

template <typename SetT>
static void launch_decode4_tile_r(int R, int XR, const uint16_t* X, int64_t m0, int rows, int64_t K, int Tk, const SetT& set, int groups, int kw, hipStream_t s) {
#define PATCH_Q4_CASE(r, xr) \
    if (R == r && XR == xr) return launch_decode4_tile<r, xr, SetT>(X, m0, rows, K, Tk, set, groups, kw, s)
    PATCH_Q4_CASE(1, 4); PATCH_Q4_CASE(2, 4); PATCH_Q4_CASE(3, 4);
    PATCH_Q4_CASE(1, 8); PATCH_Q4_CASE(2, 8); PATCH_Q4_CASE(3, 8);
#undef PATCH_Q4_CASE
}

// Strips per workgroup for a pass of `rows` rows over `strips` strips (both kernels): the R that minimises an estimate of the pass,
//     rounds(workgroups) x (x + R),
// in units of one strip's share of a wavefront's work.  x is what a workgroup spends on its X operands (it loads all of
// X whatever R is; fitted: 0.15 + 0.045 rows up to 16 rows, 1.7 for 32, 4.5 for 64 and taken from 33 on - at 4 bits per weight 64 rows of X
// are 16 times a strip's codes); rounds = workgroups / compute units, rounded up while at most two rounds are resident at
// once (then the busiest compute unit decides), with half a round for the tail beyond.  More strips per workgroup
// share X further but must not leave compute units idle: 688 strips on 256 units run as 230 workgroups of 3 (one
// round) rather than 344 of 2.  R <= 4 with two row blocks, else 3: what the registers hold.
static int q4_strips_per_group(int strips, int n_cus, int rows) {
    const int max_r = rows > 16 && rows <= 32 ? 4 : kQ4MaxR;
    const double x = rows <= 16 ? 0.15 + 0.045 * rows : rows <= 32 ? 1.7 : 4.5;
    int best = 1;
    double best_cost = 0.0;
    for (int r = 1; r <= max_r; ++r) {
        const int groups = (strips + r - 1) / r;
        const double rounds = groups <= 2 * n_cus ? (double)((groups + n_cus - 1) / n_cus) : (double)groups / n_cus + 0.5;
        const double cost = rounds * (x + r);
        if (r == 1 || cost <= best_cost) { best = r; best_cost = cost; }
    }
    return best;
}

// ------------------------------------------------------------------------------------------------------
// Batched decoding from the 4-bit storage: the workgroup of batch_kernel (gemm_batch.hip: 128 features, X through LDS, two
// wavefront groups taking the 128-column units in turn), the codes becoming operands as they are multiplied.  decode4_kernel draws
// all of X once per 16 R <= 48 features, which at 64 rows is 10 - 30 times a strip's codes; here X is drawn once per 128.
// No load is conditional: of a 2:4 tile, whose fragment lanes are 4 bytes apart, the second dword is the neighbour's (in the tile:
// positions follow the codes), and a dense tile's "positions" are its first codes; neither is used.
// ------------------------------------------------------------------------------------------------------
typedef unsigned int b4_pair_t __attribute__((ext_vector_type(2), aligned(4)));   // two dwords at a dword's alignment

struct Bt4 {
    template <int TILE>
    struct Unit {
        static constexpr int KPT = TILE / kStepCols, NT = 2 / KPT;   // steps per tile, tiles per unit
        b4_pair_t d[2][2];               // [strip][step]
        uint32_t pos[2][NT], sc[2][NT];  // [strip][tile]
        __device__ __forceinline__ void load(bt_bytes_ptr payload, bt_halves_ptr srow, int Tk, uint32_t e0, uint32_t e1, int t0, int t1, int s0, int lane) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t e = j == 0 ? e0 : e1;
                const bool sp = entry_sparse(e);
                const bt_bytes_ptr base = payload + entry_offset(e);
                const int each = sp ? 4 : 8;
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int f = (s0 + s) * KPT + (TILE == 128 ? j : 0);   // fragment
                    d[s][j] = __builtin_nontemporal_load(reinterpret_cast<const PATCH_BT_GLOBAL b4_pair_t*>(base + f * 64 * each + lane * each));
                    if (j < NT) {
                        const bt_bytes_ptr pb = base + (sp ? q4_sparse_codes(TILE) : 0) + ((s0 + s) * 64 + lane) * (2 * KPT);
                        if constexpr (KPT == 2) pos[s][j] = *reinterpret_cast<const PATCH_BT_GLOBAL uint32_t*>(pb);
                        else pos[s][j] = *reinterpret_cast<bt_halves_ptr>(pb);
                        sc[s][j] = srow[(s * Tk + (j == 0 ? t0 : t1)) * 16];
                    }
                }
            }
        }
        __device__ __forceinline__ bt_u32x4 operand(int s, int j, int h) const { return q4_dequant8(d[s][j][h], q4_bf16_to_float(sc[s][NT == 1 ? 0 : j])); }
        __device__ __forceinline__ uint32_t positions(int s, int j, int) const { return NT == 1 ? pos[s][0] >> (16 * j) : pos[s][j]; }
    };
};

// Up to kMaxMany weights that share one X; first[i] counts groups of 128 features, each weight rounded up.
struct Q4Wide {
    const uint8_t* payload[kMaxMany];
    const uint16_t* scales[kMaxMany];
    const uint32_t* table[kMaxMany];
    float* Y[kMaxMany];
    int64_t N[kMaxMany];
    int first[kMaxMany];
    int count, units;
};

template <int TILE, int RB, bool SPLIT>
__global__ __launch_bounds__(256 * bt_groups(RB)) void batch4_kernel(const uint16_t* __restrict__ X, int64_t m0, int rows, int64_t K, int Tk, const Q4Wide set) {
    uint64_t payload = reinterpret_cast<uint64_t>(set.payload[0]), scales = reinterpret_cast<uint64_t>(set.scales[0]);
    uint64_t table = reinterpret_cast<uint64_t>(set.table[0]), Y = reinterpret_cast<uint64_t>(set.Y[0]);
    int64_t N = set.N[0];
    int first = 0;
    if (set.count > 1)
#pragma unroll
        for (int i = 1; i < kMaxMany; ++i) {
            const bool here = i < set.count && (int)blockIdx.x >= set.first[i];
            payload = here ? reinterpret_cast<uint64_t>(set.payload[i]) : payload;
            scales = here ? reinterpret_cast<uint64_t>(set.scales[i]) : scales;
            table = here ? reinterpret_cast<uint64_t>(set.table[i]) : table;
            Y = here ? reinterpret_cast<uint64_t>(set.Y[i]) : Y;
            N = here ? set.N[i] : N;
            first = here ? set.first[i] : first;
        }
    batch_body<Bt4, TILE, RB, SPLIT>(X, m0, rows, K, Tk, reinterpret_cast<bt_bytes_ptr>(bt_uniform64(payload)),
                                     reinterpret_cast<bt_table_ptr>(bt_uniform64(table)), reinterpret_cast<bt_halves_ptr>(bt_uniform64(scales)),
                                     reinterpret_cast<float*>(bt_uniform64(Y)), (int64_t)bt_uniform64((uint64_t)N),
                                     (int)blockIdx.x - __builtin_amdgcn_readfirstlane(first), 0);
}

template <int TILE, bool SPLIT>
static void launch_batch4_t(const uint16_t* X, int64_t m0, int rows, int64_t K, int Tk, const Q4Wide& set, int split, hipStream_t s) {
    const dim3 grid((unsigned)set.units, (unsigned)split), block(256 * bt_groups(4));
    if (rows <= 16) hipLaunchKernelGGL((batch4_kernel<TILE, 1, SPLIT>), grid, block, 0, s, X, m0, rows, K, Tk, set);
    else if (rows <= 32) hipLaunchKernelGGL((batch4_kernel<TILE, 2, SPLIT>), grid, block, 0, s, X, m0, rows, K, Tk, set);
    else if (rows <= 48) hipLaunchKernelGGL((batch4_kernel<TILE, 3, SPLIT>), grid, block, 0, s, X, m0, rows, K, Tk, set);
    else hipLaunchKernelGGL((batch4_kernel<TILE, 4, SPLIT>), grid, block, 0, s, X, m0, rows, K, Tk, set);
}

// Up to 64 rows of X starting at row m0.  split > 1 (a set of one; at most ceil(K / 128)): K chunks, partial sums in ws (split x rows x N floats).
static void launch_batch4(const uint16_t* X, int64_t m0, int rows, int64_t K, int tile, const Q4Wide& set, int split, float* ws, hipStream_t s) {
    const int Tk = (int)(K / tile);
    if (split < 2) {
        if (tile == 128) launch_batch4_t<128, false>(X, m0, rows, K, Tk, set, 1, s);
        else launch_batch4_t<64, false>(X, m0, rows, K, Tk, set, 1, s);
        return;
    }
    Q4Wide part = set;
    part.Y[0] = ws;
    if (tile == 128) launch_batch4_t<128, true>(X, m0, rows, K, Tk, part, split, s);
    else launch_batch4_t<64, true>(X, m0, rows, K, Tk, part, split, s);
    wr_reduce(ws, (size_t)rows * (size_t)set.N[0] / 4, split, set.Y[0] + m0 * set.N[0], 0, s);
}

// ------------------------------------------------------------------------------------------------------
// Prefill-shaped product from the 4-bit storage: the structure of prefill_kernel_areg - blocks of 256
// features x 128 or 256 rows, a wavefront owns 32 features x all rows, X through two LDS stages - with the weight operands
// dequantized in registers.  A lane loads the codes of its pieces of the stored fragments one step ahead (dense: two
// 8-byte loads, fragment lanes fl and fl + 32, each holding the codes of both half-steps; 2:4: two 4-byte loads), the
// scale of its row once per tile and the position dwords once per tile; at the top of a step the codes of that step
// become bf16 operands (q4_dequant8) and the step runs as in the bf16 kernel.  The weight is read once per 128 rows of
// X, at 4 bits per kept weight, and no bf16 copy of it exists anywhere.
// ------------------------------------------------------------------------------------------------------
constexpr int kP4BN = 256;

typedef const __attribute__((address_space(1))) uint32_t* p4_g4_t;
typedef const __attribute__((address_space(1))) uint16_t* p4_g2_t;
typedef const __attribute__((address_space(1))) q4_u32x2* p4_g8_t;

// One step's codes of a wavefront.  Named by use (an array indexed by the tile type would live in scratch memory):
// half-step u multiplies the operands dequantized from (a_u, b_u); a 2:4 tile uses a_0 and a_1 only.
struct P4Codes {
    uint32_t a0, a1, b0, b1;
};

template <int TILE, int BM, bool SPLIT>
__global__ __launch_bounds__(512) void prefill4_kernel(const uint16_t* __restrict__ X, int64_t M, int64_t N, int64_t K,
                                                       const uint8_t* __restrict__ payload, const uint16_t* __restrict__ scales,
                                                       const uint32_t* __restrict__ table, int Tk_all, int tiles_n, int tiles_m,
                                                       float* __restrict__ Y) {
    constexpr int KPT = TILE / kStepCols;      // K-steps per tile: 2 or 1
    constexpr int NB = BM / 32;                // 32-row blocks: 4 or 8
    constexpr int XP = BM / 64;                // 1 KB pieces of the X tile per wavefront
    constexpr int kP4Stage = BM * 128;         // 16 or 32 KB
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fo = 32 * w;                 // first feature of the wavefront inside the block
    const int w4 = fo / TILE;              // tile row of the block its features lie in
    // block -> (n, m): one contiguous run of the grouped order (4 row blocks x all feature blocks) per XCD
    const int nblk = tiles_n * tiles_m;
    int bid = blockIdx.x;
    {
        const int per = (nblk + 7) / 8;
        const int x = bid & 7, i = bid >> 3;
        const int t = x * per + i;
        bid = (i < per && t < nblk) ? t : -1;
    }
    if (bid < 0) return;
    int bn, bm;
    {
        constexpr int GM = 4;
        const int full = (tiles_m / GM) * GM * tiles_n;
        if (bid < full) {
            const int g = bid / (GM * tiles_n), rem = bid % (GM * tiles_n);
            bn = rem / GM;
            bm = g * GM + rem % GM;
        } else {
            const int gm = tiles_m % GM, rem = bid - full;
            bn = rem / gm;
            bm = (tiles_m / GM) * GM + rem % gm;
        }
    }
    const int64_t n0 = (int64_t)bn * kP4BN, m0 = (int64_t)bm * BM;
    // N is a multiple of the tile, not necessarily of 256: a wavefront of a missing tile row works on the last live one's
    // weights (valid addresses) and stores nothing
    const int live = (int)((N - n0) / TILE) < kP4BN / TILE ? (int)((N - n0) / TILE) : kP4BN / TILE;
    const int trw = w4 < live ? w4 : live - 1;
    const int t_begin = SPLIT ? (int)((int64_t)blockIdx.y * Tk_all / gridDim.y) : 0;
    const int Tk = SPLIT ? (int)((int64_t)(blockIdx.y + 1) * Tk_all / gridDim.y) - t_begin : Tk_all;
    const uint32_t* trow = table + ((int64_t)(n0 / TILE) + trw) * Tk_all + t_begin;

    const uint8_t* xsrc[XP];
#pragma unroll
    for (int i = 0; i < XP; ++i) {
        const int c = (w + 8 * i) * 64 + lane;
        const int m = c >> 3, pp = c & 7, pl = pp ^ ((m >> 1) & 7);
        int64_t row = m0 + m;
        if (row >= M) row = M - 1;
        xsrc[i] = reinterpret_cast<const uint8_t*>(X + row * K + pl * 8 + (int64_t)t_begin * TILE);
    }
    auto load_x = [&](int ks, int stage) {
#pragma unroll
        for (int i = 0; i < XP; ++i) g2l16(xsrc[i] + (size_t)ks * 128, lds + stage * kP4Stage + (w + 8 * i) * 1024);
    };

    const int i32 = lane & 31, q = lane >> 5;
    // this lane's pieces: strip (32 w % TILE) / 16 + i32 / 16 of the tile, fragment lanes fl and fl + 32
    const int strip = (fo % TILE) / 16 + (i32 >> 4);
    const int fl = 16 * q + (i32 & 15);
    // scale of the lane's row for the first tile of this K slice; the next tile's is 16 scales on
    const uint16_t* sc = scales + q4_scale_index(((n0 + (int64_t)trw * TILE) / 16) + strip, Tk_all, t_begin, i32 & 15);
    auto load_codes = [&](P4Codes& d, uint32_t e, int j) {
        const uint8_t* tb = payload + entry_offset(e);
        if (entry_sparse(e)) {
            const uint8_t* f = tb + (size_t)(strip * KPT + j) * 256;
            d.a0 = *(p4_g4_t)(f + fl * 4);
            d.a1 = *(p4_g4_t)(f + (fl + 32) * 4);
        } else {
            const uint8_t* f = tb + (size_t)(strip * KPT + j) * 512;
            const q4_u32x2 lo = *(p4_g8_t)(f + fl * 8), hi = *(p4_g8_t)(f + (fl + 32) * 8);
            d.a0 = lo[0];
            d.a1 = lo[1];
            d.b0 = hi[0];
            d.b1 = hi[1];
        }
    };
    // per tile: the position words of fragment lanes fl and fl + 32 (mask tile 128: a dword holding both K-steps; mask
    // tile 64: 16 bits), and the scale
    auto load_tile = [&](uint32_t& d0, uint32_t& d1, uint32_t& scl, uint32_t e, int tk) {
        scl = *(p4_g2_t)(sc + (size_t)tk * 16);
        if (entry_sparse(e)) {
            const uint8_t* pb = payload + entry_offset(e) + q4_sparse_codes(TILE) + (size_t)(strip * 64 + fl) * (2 * KPT);
            if constexpr (KPT == 2) {
                d0 = *(p4_g4_t)(pb);
                d1 = *(p4_g4_t)(pb + 32 * 4);
            } else {
                d0 = *(p4_g2_t)(pb);
                d1 = *(p4_g2_t)(pb + 32 * 2);
            }
        }
    };

    f32x16 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;

    auto step_begin = [&](int ks, int pf_ks) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        load_x(pf_ks, (ks & 1) ^ 1);
    };
    auto step_mma = [&](int ks, const P4Codes& c, uint32_t p0, uint32_t p1, uint32_t sbits, int sp, int j) {
        const float scl = q4_bf16_to_float(sbits);
        A8 h0a, h0b, h1a, h1b;
        h0a.raw = q4_dequant8(c.a0, scl);
        h1a.raw = q4_dequant8(c.a1, scl);
        h0b.raw = h0a.raw;                                 // a 2:4 step does not use the second operands
        h1b.raw = h1a.raw;
        if (!sp) {
            h0b.raw = q4_dequant8(c.b0, scl);
            h1b.raw = q4_dequant8(c.b1, scl);
        }
        const uint8_t* bs = lds + (ks & 1) * kP4Stage;
        B16 xa[3], xb[3];
        auto fetch = [&](int p, int buf) {
            const int u = p / (NB / 2), b0 = 2 * (p % (NB / 2));
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                xa[buf].raw[cc] = *reinterpret_cast<const u32x4*>(bs + xs_off(32 * b0 + i32, 2 * (2 * u + cc) + q));
                xb[buf].raw[cc] = *reinterpret_cast<const u32x4*>(bs + xs_off(32 * (b0 + 1) + i32, 2 * (2 * u + cc) + q));
            }
        };
        fetch(0, 0);
        fetch(1, 1);
#pragma unroll
        for (int p = 0; p < NB; ++p) {
            if (p + 2 < NB) fetch(p + 2, (p + 2) % 3);
            const int u = p / (NB / 2), b0 = 2 * (p % (NB / 2)), buf = p % 3;
            mma_step(acc[b0], acc[b0 + 1], u ? h1a.v : h0a.v, u ? h1b.v : h0b.v, xa[buf], xb[buf], (int)((u ? p1 : p0) >> (16 * j)), sp);
        }
    };

    if constexpr (KPT == 2) {
        P4Codes c0, c1;              // codes of the even / odd step of a tile
        c0.b0 = c0.b1 = c1.b0 = c1.b1 = 0u;
        uint32_t p0 = 0u, p1 = 0u, sb = 0u, pn0 = 0u, pn1 = 0u, sbn = 0u;
        uint32_t e = trow[0];
        load_x(0, 0);
        load_codes(c0, e, 0);
        load_tile(pn0, pn1, sbn, e, 0);
        __builtin_assume(Tk > 0);
        for (int tk = 0; tk < Tk; ++tk) {
            const int more = tk + 1 < Tk ? 1 : 0;
            const uint32_t en = trow[tk + more];
            const int sp = (int)(e & 1u);
            step_begin(2 * tk, 2 * tk + 1);
            // this tile's position dwords and scale were loaded a step ago and have landed; an opaque copy, so that it does
            // not become a copy on the loop's back edge right behind the loads
            asm volatile("v_mov_b32 %0, %3\n\tv_mov_b32 %1, %4\n\tv_mov_b32 %2, %5" : "=&v"(p0), "=&v"(p1), "=&v"(sb) : "v"(pn0), "v"(pn1), "v"(sbn));
            load_codes(c1, e, 1);
            step_mma(2 * tk, c0, p0, p1, sb, sp, 0);
            step_begin(2 * tk + 1, 2 * tk + 1 + more);
            load_codes(c0, en, 0);
            load_tile(pn0, pn1, sbn, en, tk + more);
            step_mma(2 * tk + 1, c1, p0, p1, sb, sp, 1);
            e = en;
        }
    } else {
        // Mask tile 64: every step is a tile of its own, with its own scale and position words.  Steps go in pairs (the
        // buffers alternate without a copy), table entries are read two steps ahead; past the end the last step is
        // fetched again, and the second step of the last pair is skipped when the count is odd.
        const int S = Tk;
        P4Codes c0, c1;
        c0.b0 = c0.b1 = c1.b0 = c1.b1 = 0u;
        uint32_t a0 = 0u, a1 = 0u, as_ = 0u, b0_ = 0u, b1_ = 0u, bs_ = 0u;   // position words and scale of c0 / c1
        uint32_t e0 = trow[0], e1 = trow[S > 1 ? 1 : 0];
        load_x(0, 0);
        load_codes(c0, e0, 0);
        load_tile(a0, a1, as_, e0, 0);
        __builtin_assume(S > 0);
        for (int s_ = 0; s_ < S; s_ += 2) {
            const int s1 = s_ + 1 < S ? s_ + 1 : S - 1, s2 = s_ + 2 < S ? s_ + 2 : S - 1, s3 = s_ + 3 < S ? s_ + 3 : S - 1;
            const uint32_t e2 = trow[s2], e3 = trow[s3];
            step_begin(s_, s1);
            load_codes(c1, e1, 0);
            load_tile(b0_, b1_, bs_, e1, s1);
            step_mma(s_, c0, a0, a1, as_, (int)(e0 & 1u), 0);
            if (s_ + 1 < S) {
                step_begin(s_ + 1, s2);
                load_codes(c0, e2, 0);
                load_tile(a0, a1, as_, e2, s2);
                step_mma(s_ + 1, c1, b0_, b1_, bs_, (int)(e1 & 1u), 0);
            }
            e0 = e2;
            e1 = e3;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    // acc[b][i]: feature n0 + fo + 8 (i/4) + 4 q + i%4, row m0 + 32 b + i32.  The X stages are free once every wavefront
    // has left the loop: each block of 32 rows is turned through 4 KB of them and stored in whole rows
    // (store_block_rows).
    __syncthreads();
    if (w4 < live) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            store_block_rows(lds + w * 4096, acc[b], lane, Y, (SPLIT ? (int64_t)blockIdx.y * M * N : 0) + (m0 + 32 * b) * N + n0 + fo, N,
                             M - (m0 + 32 * b), 0);
    }
}

}  // namespace patch

using namespace patch;

struct patch_packed4 {
    int64_t N = 0, K = 0;
    int tile = 0, Tn = 0, Tk = 0;
    int64_t n_sparse = 0;
    size_t algorithmic_bytes = 0;   // codes + positions + scales, without alignment padding
    size_t payload_bytes = 0;
    // one allocation: payload | table | scales
    uint8_t* d_payload = nullptr;   // codes and positions
    uint32_t* d_table = nullptr;
    uint16_t* d_scales = nullptr;   // N x Tk bf16, strip-major
    std::vector<uint8_t> tile_map;  // host copy, 1 = dense
    int n_cus = 256;
};

static bool q4_aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

extern "C" {

void patch_free4(patch_packed4* P) {
    if (!P) return;
    if (P->d_payload) (void)hipFree(P->d_payload);
    delete P;
}

// The host side of a 4-bit packed weight and its device buffers, one allocation; nothing of it written yet (a tile has no alignment padding at either
// size, so that whoever fills the payload writes every byte): patch_pack4's kernel writes payload, scales and table, patch_deserialize4 copies them.
static_assert(q4_dense_tile(64) == q4_dense_codes(64) && q4_dense_tile(128) == q4_dense_codes(128) &&
              q4_sparse_tile(64) == q4_sparse_codes(64) + q4_sparse_pos(64) && q4_sparse_tile(128) == q4_sparse_codes(128) + q4_sparse_pos(128),
              "a tile with padding would have to be cleared");
static patch_status new_packed4(int64_t N, int64_t K, const uint8_t* tile_map, int tile, patch_packed4** out) {
    patch_packed4* P = new (std::nothrow) patch_packed4();
    if (!P) return PATCH_ERR_ALLOC;
    P->N = N; P->K = K; P->tile = tile;
    P->Tn = (int)(N / tile); P->Tk = (int)(K / tile);
    const size_t T = (size_t)P->Tn * (size_t)P->Tk;
    try { P->tile_map.resize(T); } catch (...) { delete P; return PATCH_ERR_ALLOC; }
    uint64_t off = 0;
    for (size_t i = 0; i < T; ++i) {
        const bool sparse = tile_map[i] == 0;
        P->tile_map[i] = sparse ? 0 : 1;
        off += sparse ? q4_sparse_tile(tile) : q4_dense_tile(tile);
        P->algorithmic_bytes += sparse ? q4_sparse_codes(tile) + q4_sparse_pos(tile) + 2 * tile : q4_dense_codes(tile) + 2 * tile;
        if (sparse) ++P->n_sparse;
    }
    P->payload_bytes = off;
    if ((off / kGranule) >> 31) { delete P; return PATCH_ERR_SHAPE; }
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
        patch_note_hip_error((int)hipGetLastError());
        delete P;
        return PATCH_ERR_HIP;
    }
    P->n_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    const size_t scales_at = (T * sizeof(uint32_t) + kGranule - 1) / kGranule * kGranule;
    if (hipMalloc(&P->d_payload, P->payload_bytes + scales_at + (size_t)N * P->Tk * sizeof(uint16_t)) != hipSuccess) {
        (void)hipGetLastError();
        patch_free4(P);
        return PATCH_ERR_ALLOC;
    }
    P->d_table = reinterpret_cast<uint32_t*>(P->d_payload + P->payload_bytes);
    P->d_scales = reinterpret_cast<uint16_t*>(P->d_payload + P->payload_bytes + scales_at);
    *out = P;
    return PATCH_OK;
}

patch_status patch_pack4(const void* W_hat, int64_t N, int64_t K, const uint8_t* tile_map, int tile, void* stream, patch_packed4** out) {
    if (!W_hat || !tile_map || !out || N <= 0 || K <= 0) return PATCH_ERR_ARG;
    if ((tile != 64 && tile != 128) || N % tile || K % tile || N / tile > (1 << 20) || K / tile > (1 << 20)) return PATCH_ERR_SHAPE;
    if (!q4_aligned16(W_hat)) return PATCH_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HostWord not_24;
    if (!not_24.valid()) return PATCH_ERR_ALLOC;
    patch_packed4* P = nullptr;
    const patch_status st = new_packed4(N, K, tile_map, tile, &P);
    if (st != PATCH_OK) return st;
    TileMapArgs map;
    uint32_t before = 0;
    for (int n_tiles = P->Tn * P->Tk, first = 0; first < n_tiles; first += kMapTiles) {
        const int n = n_tiles - first < kMapTiles ? n_tiles - first : kMapTiles;
        before = fill_map_args(&map, P->tile_map.data() + first, n, before);
        hipLaunchKernelGGL(tile == 128 ? &pack4_kernel<128> : &pack4_kernel<64>, dim3((unsigned)n), dim3(256), 0, s, map, first,
                           static_cast<const uint16_t*>(W_hat), K, P->Tk, P->d_payload, P->d_table, P->d_scales, not_24.device());
    }
    hipError_t e = hipGetLastError();
    const hipError_t e_sync = hipStreamSynchronize(s);
    if (e == hipSuccess) e = e_sync;
    if (e != hipSuccess) {
        patch_note_hip_error((int)e);
        patch_free4(P);
        return PATCH_ERR_HIP;
    }
    if (not_24.value()) {
        patch_free4(P);
        return PATCH_ERR_NOT_24;
    }
    *out = P;
    return PATCH_OK;
}

// ---- the 4-bit storage saved to and loaded from host memory (saved.h): header, tile map, codes and positions, scales
size_t patch_serialized4_bytes(const patch_packed4* P) {
    if (!P) return 0;
    return saved_round(sizeof(SavedHeader)) + saved_round(P->tile_map.size()) + saved_round(P->payload_bytes) +
           (size_t)P->N * P->Tk * sizeof(uint16_t);
}

patch_status patch_serialize4(const patch_packed4* P, void* buf, size_t bytes, void* stream) {
    if (!P || !buf) return PATCH_ERR_ARG;
    if (bytes < patch_serialized4_bytes(P)) return PATCH_ERR_SIZE;
    uint8_t* b = static_cast<uint8_t*>(buf);
    const size_t scales_bytes = (size_t)P->N * P->Tk * sizeof(uint16_t);
    const size_t map_at = saved_round(sizeof(SavedHeader)), pay_at = map_at + saved_round(P->tile_map.size());
    const size_t sc_at = pay_at + saved_round(P->payload_bytes);
    memset(b, 0, pay_at);
    memset(b + pay_at + P->payload_bytes, 0, sc_at - pay_at - P->payload_bytes);
    memcpy(b + map_at, P->tile_map.data(), P->tile_map.size());
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e = hipMemcpyAsync(b + pay_at, P->d_payload, P->payload_bytes, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(b + sc_at, P->d_scales, scales_bytes, hipMemcpyDeviceToHost, s);
    const hipError_t e_sync = hipStreamSynchronize(s);
    if (e == hipSuccess) e = e_sync;
    if (e != hipSuccess) { patch_note_hip_error((int)e); return PATCH_ERR_HIP; }
    SavedHeader h = {};
    memcpy(h.magic, kSavedMagic4, 8);
    h.layout = kSavedLayout;
    h.tile = (uint32_t)P->tile;
    h.N = P->N;
    h.K = P->K;
    h.map_bytes = P->tile_map.size();
    h.payload_bytes = P->payload_bytes;
    h.aux_bytes = scales_bytes;
    h.checksum = fnv1a(b + sc_at, scales_bytes, fnv1a(b + pay_at, P->payload_bytes, fnv1a(b + map_at, P->tile_map.size(), kFnvBasis)));
    memcpy(b, &h, sizeof(h));
    return PATCH_OK;
}

patch_status patch_deserialize4(const void* buf, size_t bytes, void* stream, patch_packed4** out) {
    if (!buf || !out) return PATCH_ERR_ARG;
    if (bytes < saved_round(sizeof(SavedHeader))) return PATCH_ERR_SIZE;
    const uint8_t* b = static_cast<const uint8_t*>(buf);
    SavedHeader h;
    memcpy(&h, b, sizeof(h));
    if (memcmp(h.magic, kSavedMagic4, 8) != 0 || h.layout != kSavedLayout) return PATCH_ERR_ARG;
    if (h.N <= 0 || h.K <= 0) return PATCH_ERR_ARG;
    if ((h.tile != 64 && h.tile != 128) || h.N % h.tile || h.K % h.tile || h.N / h.tile > (1 << 20) || h.K / h.tile > (1 << 20))
        return PATCH_ERR_SHAPE;
    const uint64_t Tk = (uint64_t)(h.K / h.tile), T = (uint64_t)(h.N / h.tile) * Tk;
    if (h.map_bytes != T || h.aux_bytes != (uint64_t)h.N * Tk * sizeof(uint16_t)) return PATCH_ERR_ARG;
    const size_t map_at = saved_round(sizeof(SavedHeader)), pay_at = map_at + saved_round((size_t)T);
    if (bytes < pay_at || h.payload_bytes > bytes - pay_at) return PATCH_ERR_SIZE;
    const size_t sc_at = pay_at + saved_round((size_t)h.payload_bytes);
    if (bytes < sc_at || h.aux_bytes > bytes - sc_at) return PATCH_ERR_SIZE;
    for (uint64_t i = 0; i < T; ++i)
        if (b[map_at + i] > 1) return PATCH_ERR_ARG;
    if (fnv1a(b + sc_at, (size_t)h.aux_bytes, fnv1a(b + pay_at, (size_t)h.payload_bytes, fnv1a(b + map_at, (size_t)T, kFnvBasis))) != h.checksum)
        return PATCH_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    patch_packed4* P = nullptr;
    const patch_status st = new_packed4(h.N, h.K, b + map_at, (int)h.tile, &P);
    if (st != PATCH_OK) return st;
    if (P->payload_bytes != h.payload_bytes) {   // the map decides the size: a header that disagrees is not ours
        patch_free4(P);
        return PATCH_ERR_ARG;
    }
    std::vector<uint32_t> table;
    try { table.resize(T); } catch (...) { patch_free4(P); return PATCH_ERR_ALLOC; }
    uint64_t off = 0;
    for (size_t i = 0; i < T; ++i) {
        table[i] = make_entry(off, !P->tile_map[i]);
        off += P->tile_map[i] ? q4_dense_tile(P->tile) : q4_sparse_tile(P->tile);
    }
    hipError_t e = hipMemcpyAsync(P->d_table, table.data(), T * sizeof(uint32_t), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(P->d_payload, b + pay_at, P->payload_bytes, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(P->d_scales, b + sc_at, (size_t)h.aux_bytes, hipMemcpyHostToDevice, s);
    const hipError_t e_sync = hipStreamSynchronize(s);   // the caller's buffer is free to go when the call returns
    if (e == hipSuccess) e = e_sync;
    if (e != hipSuccess) {
        patch_note_hip_error((int)e);
        patch_free4(P);
        return PATCH_ERR_HIP;
    }
    *out = P;
    return PATCH_OK;
}

patch_status patch_unpack4(const patch_packed4* P, void* W_deq, void* codes, void* scales, void* stream) {
    if (!P || (!W_deq && !codes && !scales)) return PATCH_ERR_ARG;
    if ((W_deq && !q4_aligned16(W_deq)) || (scales && (reinterpret_cast<uintptr_t>(scales) & 1u))) return PATCH_ERR_ARG;
    hipLaunchKernelGGL(P->tile == 128 ? &unpack4_kernel<128> : &unpack4_kernel<64>, dim3((unsigned)(P->Tn * P->Tk)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), P->d_payload, P->d_scales, P->d_table, P->Tk, P->K, static_cast<uint16_t*>(W_deq),
                       static_cast<int8_t*>(codes), static_cast<uint16_t*>(scales));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { patch_note_hip_error((int)e); return PATCH_ERR_HIP; }
    return PATCH_OK;
}

// What the choices below go by: `count` weights of N features and K columns together (a single weight's K may be split over ws_bytes of
// workspace, 0 = none), f = share of 2:4 tiles.
struct Q4Shape { int count, strips, groups128; int64_t N, K; int tile, n_cus; double f; size_t ws_bytes; };

static Q4Shape q4_shape(const patch_packed4* const* P, int count, size_t ws_bytes) {
    Q4Shape d = {count, 0, 0, 0, P[0]->K, P[0]->tile, P[0]->n_cus, 0.0, count == 1 ? ws_bytes : 0};
    double sparse = 0.0, tiles = 0.0;
    for (int i = 0; i < count; ++i) {
        d.strips += (int)(P[i]->N / kStripRows);
        d.groups128 += (int)((P[i]->N + kBtFeatures - 1) / kBtFeatures);
        d.N += P[i]->N;
        sparse += (double)P[i]->n_sparse;
        tiles += (double)P[i]->Tn * P[i]->Tk;
    }
    d.f = sparse / tiles;
    return d;
}

// A pass of `rows` rows (at most 64) over all weights: the strip kernel or batch4_kernel, and in how many K chunks.  Both are priced, in us with
// steps = 64-column steps, fitted by row range to launches of weights and sets, both mask tiles, f = 0, 1/2 and 1 (strip: 42 shapes, 25 row counts, 630 - 1764
// launches per line, rms error 7 - 8 %; batch: 36 shapes, 14 row counts, 650 - 4100 launches per line, 5 - 8 %):
//   strip   base + turns x (per_strip R + constant + per_row rows) x 0.05 x steps x (1 + sparse (f - 1/2)); R = strips per workgroup, turns = 1 up to one
//           workgroup per compute unit, beyond over x ((1 - whole) share + whole ceil(share) + late where share > 2), share = workgroups / compute units:
//           the unit with the most workgroups decides most of it, and two are resident.  (By share alone, launches just past a whole number were
//           estimated up to 29 % short and those just below it up to 30 % long.)
//   batch   base + (1 + round (rounds - 1)) x steps / chunks x (step + per_row rows) x (1 + fill min(1, workgroups / compute units)) x (tile64 on mask
//           tile 64: two scales and position loads per unit) x (1 + sparse (f - 1/2)); a split 2.7 for the second launch and its partial sums twice at
//           5 TB/s
// The cheaper one is taken, the batch kernel up to 8 rows if it is 0.4 ahead, up to 16 also 0.2 behind (its K chunks are estimated that much long there:
// 4096 x 11008, f = 1, 12 rows 10.9, measured 10.8, the strip kernel 10.9 and 13.0).  Over those 42 shapes that is 0.02 - 0.27 % slower, by row range and mask tile,
// than the faster of the two always (by share alone, and the batch kernel to be 0.8 ahead, up to 8 rows 2.5, up to 12 2.2: 0.1 - 0.9 %).
// Measured, strip / batch, f = 1/2, mask tile 128: gate and up of 4096 / 11008 at 1 / 16 / 32 / 64 rows (13.7 / 19.0, 16.6 / 19.5, 23.2 / 22.2, 40.1 / 28.3), of 5120 /
// 13824 (20.0 / 23.8, 26.6 / 23.6, 34.2 / 27.5, 70.4 / 35.1); three 4096 x 4096 (8.6 / 19.2, 10.3 / 19.2, 13.8 / 21.6, 21.6 / 27.0).
struct Q4StripPrice { int rows; double base, per_strip, constant, per_row, over, whole, sparse, late; };
constexpr Q4StripPrice kQ4StripPrice[] = {{8, 3.119, 0.522, 0.041, 0.029, 0.966, 0.777, -0.314, -0.172}, {16, 2.971, 0.452, 0.076, 0.045, 0.95, 0.888, -0.284, -0.131},
                                          {32, 3.087, 0.528, 0.238, 0.046, 1.029, 0.485, -0.178, 0.395}, {48, 3.244, 0.508, 0.341, 0.052, 1.023, 0.867, -0.108, 0.116},
                                          {64, 3.43, 0.546, 0.517, 0.052, 1.039, 0.871, -0.083, 0.088}};
constexpr Q4StripPrice kQ4TilePrice = {8, 3.108, 0.531, -0.059, 0.028, 1.016, 0.579, -0.306, 0.043};   // decode4_tile_kernel: mask tile 128, up to 8 rows
struct Q4BatchPrice { int rows; double base, step, per_row, fill, tile64, sparse, round; };
constexpr Q4BatchPrice kQ4BatchPrice[] = {{16, 2.7, 0.2204, 0.0001, 0.17, 1.12, -0.24, 0.53}, {32, 3.0, 0.2487, 0.0003, 0.15, 1.11, -0.21, 0.57}, {64, 3.6, 0.217, 0.0019, 0.15, 1.10, -0.20, 1.05}};

struct Q4Plan { bool wide; int chunks; double us; };
static Q4Plan q4_pass_plan(const Q4Shape& d, int rows) {
    const double steps = (double)d.K / kStepCols;
    const Q4StripPrice* p = d.tile == 128 && rows <= 8 ? &kQ4TilePrice : kQ4StripPrice;
    while (rows > p->rows) ++p;
    const int R = q4_strips_per_group(d.strips, d.n_cus, rows);
    const int groups = (d.strips + R - 1) / R;
    const double turns = groups <= d.n_cus ? 1.0 : p->over * ((1.0 - p->whole) * groups / d.n_cus + p->whole * ((groups + d.n_cus - 1) / d.n_cus) + (groups > 2 * d.n_cus ? p->late : 0.0));
    const Q4Plan strip = {false, 1, p->base + turns * (p->per_strip * R + p->constant + p->per_row * rows) * 0.05 * steps * (1.0 + p->sparse * (d.f - 0.5))};
    const Q4BatchPrice* b = kQ4BatchPrice;
    while (rows > b->rows) ++b;
    const size_t fit = d.ws_bytes / ((size_t)rows * (size_t)d.N * sizeof(float));
    Q4Plan wide = {true, 1, 0.0};
    for (int c = 1; c == 1 || (c <= 8 && (size_t)c <= fit && d.groups128 * c <= d.n_cus && c * 512 <= d.K); ++c) {
        const int wg = d.groups128 * c, rounds = (wg + d.n_cus - 1) / d.n_cus;
        const double fill = wg < d.n_cus ? (double)wg / d.n_cus : 1.0;
        const double us = b->base + (1.0 + b->round * (rounds - 1)) * steps / c * (b->step + b->per_row * rows) * (1.0 + b->fill * fill) * (d.tile == 64 ? b->tile64 : 1.0) *
                              (1.0 + b->sparse * (d.f - 0.5)) +
                          (c > 1 ? 2.7 + 2.0 * c * rows * (double)d.N * 4.0 / 5.0e6 : 0.0);
        if (c == 1 || us < wide.us) wide = Q4Plan{true, c, us};
    }
    return wide.us + (rows <= 8 ? 0.4 : rows <= 16 ? -0.2 : 0.0) < strip.us ? wide : strip;
}

static patch_status q4_passes(const void* X, int64_t M, const patch_packed4* const* P, void* const* Y, int count, float* ws, size_t ws_bytes,
                              hipStream_t s, const Q4Plan* asked = nullptr);

patch_status patch_gemm4_many(const void* X, int64_t M, const patch_packed4* const* P, void* const* Y, int count, void* stream) {
    if (!X || !P || !Y || M < 0 || count < 1 || count > PATCH_MAX_MANY) return PATCH_ERR_ARG;
    static_assert(PATCH_MAX_MANY == kMaxMany, "header and kernels disagree");
    if (!q4_aligned16(X)) return PATCH_ERR_ARG;
    for (int i = 0; i < count; ++i) {
        if (!P[i] || !Y[i] || !q4_aligned16(Y[i])) return PATCH_ERR_ARG;
        if (P[i]->K != P[0]->K || P[i]->tile != P[0]->tile) return PATCH_ERR_SHAPE;
    }
    if (M == 0) return PATCH_OK;
    return q4_passes(X, M, P, Y, count, nullptr, 0, static_cast<hipStream_t>(stream));
}

// Passes of up to 64 rows over all weights, which share X (checked by the callers): the strip kernel or batch4_kernel, whichever is
// estimated faster, or the one `asked` for.  A single weight may split K over a workspace.
static patch_status q4_passes(const void* X, int64_t M, const patch_packed4* const* P, void* const* Y, int count, float* ws, size_t ws_bytes,
                              hipStream_t s, const Q4Plan* asked) {
    const patch_packed4* P0 = P[0];
    const int total = P0->Tk * (P0->tile / kStepCols);
    int first[kMaxMany], total_strips = 0;
    for (int i = 0; i < count; ++i) {
        first[i] = total_strips;
        total_strips += (int)(P[i]->N / kStripRows);
    }
    Q4Wide wide = {};
    for (int i = 0; i < count; ++i) {
        wide.payload[i] = P[i]->d_payload;
        wide.scales[i] = P[i]->d_scales;
        wide.table[i] = P[i]->d_table;
        wide.Y[i] = static_cast<float*>(Y[i]);
        wide.N[i] = P[i]->N;
        wide.first[i] = wide.units;
        wide.units += (int)((P[i]->N + kBtFeatures - 1) / kBtFeatures);
    }
    wide.count = count;
    const Q4Shape shape = q4_shape(P, count, ws_bytes);
    // One launch per pass of up to 64 rows, R strips per workgroup (q4_strips_per_group).
    auto run = [&](const auto& set) {
        for (int64_t m0 = 0; m0 < M; m0 += kQ4Rows) {
            const int rows = (int)(M - m0 < kQ4Rows ? M - m0 : kQ4Rows);
            const Q4Plan plan = asked ? *asked : q4_pass_plan(shape, rows);
            if (plan.wide) {
                launch_batch4(static_cast<const uint16_t*>(X), m0, rows, P0->K, P0->tile, wide, plan.chunks, ws, s);
                continue;
            }
            const int RB = (rows + 15) / 16;
            const int R = q4_strips_per_group(total_strips, P0->n_cus, rows);
            const int groups = (total_strips + R - 1) / R;
            // wavefronts per workgroup: about 4 steps each, at least 4, at most 16 (8 with many registers); with more
            // workgroups than compute units half of that, so that two workgroups share a compute unit (its registers
            // hold 16 of these wavefronts) instead of running one after the other
            int kw = (total + 3) / 4;
            if (kw > q4_max_waves(R, RB)) kw = q4_max_waves(R, RB);
            if (groups > P0->n_cus && kw > 8) kw = 8;
            kw = (kw + 3) / 4 * 4;   // sum_in_order
            if (P0->tile == 128 && rows <= 8) {
                // wavefronts per workgroup: 16 per compute unit in one, two or more workgroups, at least two tiles each (22 shapes, 5 row counts, f = 0, 1/2, 1:
                // 1.7 % behind the best of 15 pairs of strips and wavefronts on average, 10 % at most)
                kw = groups <= P0->n_cus ? 16 : groups <= 2 * P0->n_cus ? 8 : 4;
                while (kw > 4 && 2 * kw > P0->Tk) kw /= 2;
                launch_decode4_tile_r(R, rows <= 4 ? 4 : 8, static_cast<const uint16_t*>(X), m0, rows, P0->K, P0->Tk, set, groups, kw, s);
                continue;
            }
            if (P0->tile == 128) launch_decode4_r<128>(R, RB, static_cast<const uint16_t*>(X), m0, rows, P0->K, P0->Tk, set, groups, kw, s);
            else launch_decode4_r<64>(R, RB, static_cast<const uint16_t*>(X), m0, rows, P0->K, P0->Tk, set, groups, kw, s);
        }
    };
    auto fill = [&](auto& set) {
        for (int i = 0; i < count; ++i) {
            set.payload[i] = P[i]->d_payload;
            set.scales[i] = P[i]->d_scales;
            set.table[i] = P[i]->d_table;
            set.Y[i] = static_cast<float*>(Y[i]);
            set.N[i] = P[i]->N;
            set.first[i] = first[i];
        }
        set.count = count;
        set.total = total_strips;
    };
    // the fewer kernel arguments the better: a set of one, of up to three (q / k / v, gate / up), of up to eight
    if (count == 1) {
        run(Q4One{P0->d_payload, P0->d_scales, P0->d_table, static_cast<float*>(Y[0]), P0->N});
    } else if (count <= 3) {
        Q4Set<3> set = {};
        fill(set);
        run(set);
    } else {
        Q4Set<kMaxMany> set = {};
        fill(set);
        run(set);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { patch_note_hip_error((int)e); return PATCH_ERR_HIP; }
    return PATCH_OK;
}

patch_status patch_gemm4(const void* X, int64_t M, const patch_packed4* P, void* Y, void* stream) {
    return patch_gemm4_ex(X, M, P, Y, nullptr, 0, stream);
}

// Passes of up to 64 rows or the prefill-shaped kernel?  Both sides are estimated from measured rates, as for the bf16 kernels:
//   passes           q4_pass_plan's estimate of a full pass, and of the last one by its rows
//   prefill kernels  base + start fill + round (rounds - 1) + rounds x steps per workgroup x (t0 + t1 fill) x (tile64 on mask tile 64) x (1 + sparse (f - 1/2)),
//                    fill = min(1, workgroups / compute units), + for a split second x (3 + (2 split + 1) M N 4 B / 8.3 TB/s); splits of at most 8
//                    slices of at least 512 columns.  prefill4_kernel in blocks of 128 and of 256 rows (which converts the same codes for twice the
//                    rows): fitted to 9072 and 9630 launches of 24 weights at 17 - 400 rows, both mask tiles, f = 0, 1/2 and 1 (rms error 4 %).
//                    prefill4_kgroups_kernel (128 rows; its workgroup starts later and adds two halves at the end, and its steps are a third
//                    shorter): 3012 launches of 13 weights from 896 x 896 to 13824 x 5120 at 40 - 4096 rows (4.7 %), and has to be 2 % ahead.
// Held against all 8249 launches, with a workspace: 0.94 of the time that prefill4_kernel alone chose, one of 772 calls 1.4 % more; without: 0.79 and
// none.  (Passes are given up by prefill4_kernel's price alone, as before: 1024 x 8192 at 193 rows without a workspace, four passes 101 us, would take
// about 85.)  prefill4_kernel stays ahead on few steps per workgroup (1024 x 1024 at 200 rows, f = 1: 12.2 us against 14.9; 4864 x 896 at 2048 rows 24.5 and 30.8).
// Returns the split to launch the prefill kernel with (and which), or 0 for passes.
enum Q4PrefillKernel { kQ4Rows128, kQ4Rows256, kQ4Groups };
struct Q4PrefillPrice { int bm; double base, start, round, t0, t1, tile64, sparse, second; };
constexpr Q4PrefillPrice kQ4PrefillPrice[] = {{128, 4.6, 0.0, 0.0, 0.766, 0.076, 1.065, -0.30, 1.0}, {256, 6.1, 0.0, 0.0, 1.22, 0.142, 1.054, -0.387, 1.0},
                                              {128, 8.1, 1.5, 4.1, 0.489, 0.142, 1.023, -0.255, 0.91}};

static int q4_prefill_split(int64_t M, const Q4Shape& d, Q4PrefillKernel* kernel, int* tail) {
    *kernel = kQ4Rows128;
    *tail = 0;
    if (M <= 16) return 0;
    const int kpt = d.tile / kStepCols, Tk = (int)(d.K / d.tile);
    const int64_t full = M / kQ4Rows;
    const int rest = (int)(M % kQ4Rows);
    const double passes_us = (full ? (double)full * q4_pass_plan(d, kQ4Rows).us : 0.0) + (rest ? q4_pass_plan(d, rest).us : 0.0);
    const size_t per_slice = (size_t)M * (size_t)d.N * sizeof(float);
    const size_t fit = d.ws_bytes / per_slice;
    int best_split = 1;
    double best = 0.0;
    const auto take = [&](Q4PrefillKernel k) {
        const Q4PrefillPrice& p = kQ4PrefillPrice[k];
        const int64_t blocks = ((d.N + kP4BN - 1) / kP4BN) * ((M + p.bm - 1) / p.bm);
        for (int sp = 1; sp == 1 || (sp <= 8 && (size_t)sp <= fit && sp * 512 <= d.K); ++sp) {
            const int64_t wgs = blocks * sp, rounds = (wgs + d.n_cus - 1) / d.n_cus;
            const double fill = wgs < d.n_cus ? (double)wgs / d.n_cus : 1.0;
            int steps = ((Tk + sp - 1) / sp) * kpt;
            if (k == kQ4Groups) steps = (steps + 1) / 2 * 2;   // units of two
            double us = p.base + p.start * fill + p.round * (double)(rounds - 1) + (double)(rounds * steps) * (p.t0 + p.t1 * fill) * (d.tile == 64 ? p.tile64 : 1.0) * (1.0 + p.sparse * (d.f - 0.5));
            if (sp > 1) us += p.second * (3.0 + (2.0 * sp + 1.0) * (double)per_slice / 8.3e6);
            if (k == kQ4Groups) us *= 1.02;
            if (best == 0.0 || us < best) { best = us; best_split = sp; *kernel = k; }
        }
    };
    take(kQ4Rows128);
    take(kQ4Rows256);
    if (best >= passes_us) return 0;
    if (d.K > kKgMaxK) return best_split;
    take(kQ4Groups);
    // ... and, with a workspace, the blocks beyond a multiple of the compute units in a launch of their own, K in slices that fill the chip at most once and are
    // summed by a third: up to four full rounds, up to half a round left, 4 % and 4 us below.  60 launches of 7 weights at 640 - 4200 rows: 0.908 of the
    // best undivided launch over all, none slower; us, undivided -> so: 11008 x 4096, f = 1/2, 800 rows (301 blocks) 94.1 -> 83.4, 1536 rows (516) 144.3 -> 131.6;
    // 4096 x 11008, 2100 rows (272) 223.8 -> 166.5; half a round left gains least (4096 x 4096, 3000 rows, 384 blocks 92.5 and 96.5: not taken).
    const Q4PrefillPrice& p = kQ4PrefillPrice[kQ4Groups];
    const int64_t blocks = ((d.N + kP4BN - 1) / kP4BN) * ((M + p.bm - 1) / p.bm), whole = blocks / d.n_cus, t = blocks % d.n_cus;
    if (whole < 1 || whole > 4 || t == 0 || 2 * t > d.n_cus) return best_split;
    const double step = (d.tile == 64 ? p.tile64 : 1.0) * (1.0 + p.sparse * (d.f - 0.5));
    for (int sp = 2; sp <= 8 && sp * t <= d.n_cus && sp * 512 <= d.K && (size_t)sp * (size_t)t * kKgSlotBytes <= d.ws_bytes; ++sp) {
        const double fill = (double)(sp * t) / d.n_cus;
        const int steps = (((Tk + sp - 1) / sp) * kpt + 1) / 2 * 2;
        const double body = p.base + p.start + p.round * (double)(whole - 1) + (double)(whole * Tk * kpt) * (p.t0 + p.t1) * step;
        const double last = p.base + p.start * fill + (double)steps * (p.t0 + p.t1 * fill) * step + p.second * (3.0 + (2.0 * sp + 1.0) * (double)t * (double)kKgSlotBytes / 8.3e6);
        const double us = 1.04 * (body + last) + 4.0;
        if (us < best) { best = us; best_split = sp; *kernel = kQ4Groups; *tail = (int)t; }
    }
    return best_split;
}

// Test hook (kernels.h)
int patch_test_schedule4(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes, int* kernel, int* chunks) {
    if (!N || !kernel || !chunks || M < 1 || count < 1 || count > kMaxMany || (tile != 64 && tile != 128) || K < tile || K % tile || sparse_pct < 0 || sparse_pct > 100) return -1;
    Q4Shape d = {count, 0, 0, 0, K, tile, 256, 0.01 * sparse_pct, 0};
    for (int i = 0; i < count; ++i) {
        if (N[i] < tile || N[i] % tile) return -1;
        d.strips += (int)(N[i] / kStripRows);
        d.groups128 += (int)((N[i] + kBtFeatures - 1) / kBtFeatures);
        d.N += N[i];
    }
    if (count == 1 && ws_bytes >= 2 * (size_t)M * (size_t)d.N * sizeof(float)) d.ws_bytes = ws_bytes;
    Q4PrefillKernel which;
    int tail;
    if (const int split = count == 1 ? q4_prefill_split(M, d, &which, &tail) : 0) {
        kernel[0] = tail ? 5 : 2 + which;
        chunks[0] = split;
        return 1;
    }
    if (M > 8 * kQ4Rows) return -1;
    int n = 0;
    for (int64_t m0 = 0; m0 < M; m0 += kQ4Rows, ++n) {
        const Q4Plan plan = q4_pass_plan(d, (int)(M - m0 < kQ4Rows ? M - m0 : kQ4Rows));
        kernel[n] = plan.wide ? 1 : 0;
        chunks[n] = plan.chunks;
    }
    return n;
}

// One prefill-shaped launch; split > 1: K slices, partial sums in ws (split x M x N floats); tail > 0: of the last blocks alone (launch_prefill4_kgroups).
static patch_status q4_prefill(const uint16_t* X, int64_t M, const patch_packed4* P, float* Y, int split, Q4PrefillKernel kernel, int tail, float* ws, hipStream_t s) {
    const int bm = kernel == kQ4Rows256 ? 256 : 128;
    const int tiles_n = (int)((P->N + kP4BN - 1) / kP4BN), tiles_m = (int)((M + bm - 1) / bm);
    const int grid = ((tiles_n * tiles_m + 7) / 8) * 8;
    const int lds_bytes = 2 * bm * 128;
    auto launch = [&](auto whole, auto sliced) {
        if (split == 1) {
            hipLaunchKernelGGL(whole, dim3(grid), dim3(512), lds_bytes, s, X, M, P->N, P->K, P->d_payload, P->d_scales, P->d_table, P->Tk, tiles_n,
                               tiles_m, Y);
        } else {
            hipLaunchKernelGGL(sliced, dim3(grid, split), dim3(512), lds_bytes, s, X, M, P->N, P->K, P->d_payload, P->d_scales, P->d_table, P->Tk,
                               tiles_n, tiles_m, ws);
            wr_reduce(ws, (size_t)M * (size_t)P->N / 4, split, Y, 0, s);
        }
    };
    if (kernel == kQ4Groups) {
        launch_prefill4_kgroups({X, M, P->N, P->K, P->tile, P->Tk, P->d_payload, P->d_scales, P->d_table, Y}, split, tail, ws, s);
        if (split > 1 && tail == 0) wr_reduce(ws, (size_t)M * (size_t)P->N / 4, split, Y, 0, s);
    } else if (P->tile == 128 && bm == 128) launch(prefill4_kernel<128, 128, false>, prefill4_kernel<128, 128, true>);
    else if (P->tile == 128) launch(prefill4_kernel<128, 256, false>, prefill4_kernel<128, 256, true>);
    else if (bm == 128) launch(prefill4_kernel<64, 128, false>, prefill4_kernel<64, 128, true>);
    else launch(prefill4_kernel<64, 256, false>, prefill4_kernel<64, 256, true>);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) { patch_note_hip_error((int)err); return PATCH_ERR_HIP; }
    return PATCH_OK;
}

patch_status patch_gemm4_ex(const void* X, int64_t M, const patch_packed4* P, void* Y, void* workspace, size_t workspace_bytes,
                            void* stream) {
    if (!X || !P || !Y || M < 0) return PATCH_ERR_ARG;
    if (!q4_aligned16(X) || !q4_aligned16(Y) || (workspace && !q4_aligned16(workspace))) return PATCH_ERR_ARG;
    if (M == 0) return PATCH_OK;
    const bool ws = workspace && workspace_bytes >= 2 * (size_t)M * (size_t)P->N * sizeof(float);
    float* const part = ws ? static_cast<float*>(workspace) : nullptr;
    const size_t part_bytes = ws ? workspace_bytes : 0;
    Q4PrefillKernel kernel;
    int tail;
    const int split = q4_prefill_split(M, q4_shape(&P, 1, part_bytes), &kernel, &tail);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (split == 0) return q4_passes(X, M, &P, &Y, 1, part, part_bytes, s);
    return q4_prefill(static_cast<const uint16_t*>(X), M, P, static_cast<float*>(Y), split, kernel, tail, part, s);
}

// Test hook (kernels.h)
int patch_test_gemm4(const void* X, int64_t M, const patch_packed4* const* P, void* const* Y, int count, int kernel, int chunks,
                              void* workspace, size_t workspace_bytes, void* stream) {
    if (!X || !P || !Y || M < 1 || count < 1 || count > kMaxMany || kernel < 0 || kernel > 5 || !q4_aligned16(X)) return PATCH_ERR_ARG;
    for (int i = 0; i < count; ++i) {
        if (!P[i] || !Y[i] || !q4_aligned16(Y[i])) return PATCH_ERR_ARG;
        if (P[i]->K != P[0]->K || P[i]->tile != P[0]->tile) return PATCH_ERR_SHAPE;
    }
    const int longest = kernel == 1 ? (int)((P[0]->K + kBtUnit - 1) / kBtUnit) : kernel == 0 ? 1 : P[0]->Tk;
    const int64_t rows = kernel == 1 && M > kQ4Rows ? kQ4Rows : M;
    if (chunks < 1 || chunks > longest || (count > 1 && (chunks > 1 || kernel > 1))) return PATCH_ERR_ARG;
    const int64_t blocks = ((P[0]->N + 255) / 256) * ((M + 127) / 128);
    const int tail = kernel == 5 ? (int)(blocks % P[0]->n_cus) : 0;
    if (kernel == 5) {
        if (chunks < 2 || blocks < P[0]->n_cus || tail == 0) return PATCH_ERR_ARG;
        if (!workspace || !q4_aligned16(workspace) || workspace_bytes < (size_t)chunks * (size_t)tail * kKgSlotBytes) return PATCH_ERR_SIZE;
    } else if (chunks > 1 && (!workspace || !q4_aligned16(workspace) || workspace_bytes < (size_t)chunks * (size_t)rows * (size_t)P[0]->N * sizeof(float))) {
        return PATCH_ERR_SIZE;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (kernel >= 4 && P[0]->K > kKgMaxK) return PATCH_ERR_SHAPE;
    if (kernel > 1)
        return q4_prefill(static_cast<const uint16_t*>(X), M, P[0], static_cast<float*>(Y[0]), chunks, kernel == 5 ? kQ4Groups : (Q4PrefillKernel)(kernel - 2), tail,
                          static_cast<float*>(workspace), s);
    const Q4Plan plan = {kernel == 1, chunks, 0.0};
    return q4_passes(X, M, P, Y, count, static_cast<float*>(workspace), workspace_bytes, s, &plan);
}

patch_status patch_pack_from4(const patch_packed4* P4, void* stream, patch_packed** out) {
    if (!P4 || !out) return PATCH_ERR_ARG;
    uint16_t* W_deq = nullptr;
    if (hipMalloc(&W_deq, (size_t)P4->N * (size_t)P4->K * sizeof(uint16_t)) != hipSuccess) {
        (void)hipGetLastError();
        return PATCH_ERR_ALLOC;
    }
    patch_status st = patch_unpack4(P4, W_deq, nullptr, nullptr, stream);
    // patch_pack runs on the same stream behind the dequantization and waits for the stream before it returns
    if (st == PATCH_OK) st = patch_pack(W_deq, P4->N, P4->K, P4->tile_map.data(), P4->tile, stream, out);
    else (void)hipStreamSynchronize(static_cast<hipStream_t>(stream));
    (void)hipFree(W_deq);
    return st;
}

size_t patch_packed4_bytes(const patch_packed4* P) { return P ? P->algorithmic_bytes : 0; }

patch_status patch_packed4_dims(const patch_packed4* P, int64_t* N, int64_t* K, int* tile, int64_t* n_sparse_tiles) {
    if (!P) return PATCH_ERR_ARG;
    if (N) *N = P->N;
    if (K) *K = P->K;
    if (tile) *tile = P->tile;
    if (n_sparse_tiles) *n_sparse_tiles = P->n_sparse;
    return PATCH_OK;
}

}  // extern "C"
