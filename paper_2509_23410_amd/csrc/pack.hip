// Mask merge, compression and decompression kernels (gfx950).
//
// Compression follows Appendix A of the paper (compress a mixed dense / 2:4 weight for a given tile size);
// the mask merge follows the last lines of Algorithm 1 / Eq. 4 with hard masks.  The byte layout written
// here is described in layout.h.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include "kernels.h"
#include "layout.h"
#include "map_args.h"

namespace patch {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ small data as kernel arguments
// Eight bytes to eight bits, nonzero = 1, the first byte lowest
static inline uint64_t nonzero_bits(const uint8_t* bytes) {
    constexpr uint64_t low7 = 0x7f7f7f7f7f7f7f7full;
    uint64_t x;
    memcpy(&x, bytes, 8);
    x = (((x & low7) + low7) | x) & ~low7;            // the top bit of every nonzero byte
    return ((x >> 7) * 0x0102040810204080ull) >> 56;   // byte i's bit to bit 56 + i, without carries
}

// (on the way of every call that has a map: 19456 tiles byte by byte took 18.5 us, eight at a time 3.6)
uint32_t fill_map_args(TileMapArgs* a, const uint8_t* map, int n, uint32_t before) {
    for (int g = 0; 64 * g < n; ++g) {
        const int here = n - 64 * g < 64 ? n - 64 * g : 64;
        uint64_t bits = 0;
        int i = 0;
        for (; i + 8 <= here; i += 8) bits |= nonzero_bits(map + 64 * g + i) << i;
        for (; i < here; ++i) bits |= (uint64_t)(map[64 * g + i] != 0) << i;
        a->g[g].dense[0] = (uint32_t)bits;
        a->g[g].dense[1] = (uint32_t)(bits >> 32);
        a->g[g].before = before;
        before += (uint32_t)__builtin_popcountll(bits);
    }
    return before;
}

constexpr int kPutWords = 896;
struct PutWords { uint32_t w[kPutWords]; };
__global__ __launch_bounds__(64) void put_words_kernel(const PutWords words, uint32_t* __restrict__ dst, int n) {
    for (int i = threadIdx.x; i < n; i += 64) dst[i] = words.w[i];
}

void launch_put_words(uint32_t* dst, const uint32_t* src, size_t n, hipStream_t stream) {
    for (size_t at = 0; at < n; at += kPutWords) {
        PutWords words;
        const int part = (int)(n - at < (size_t)kPutWords ? n - at : (size_t)kPutWords);
        memcpy(words.w, src + at, part * sizeof(uint32_t));
        hipLaunchKernelGGL(put_words_kernel, dim3(1), dim3(64), 0, stream, words, dst + at, part);
    }
}

// ------------------------------------------------------------------ mask merge
// A wavefront and step: up to 512 consecutive elements of a row, 8 per lane (16 bytes of W, 8 bytes of mask), whose tiles are at most eight consecutive
// bits of the map; or, where a row is at most 256 long (ROW_LANES < 64 lanes of 8 elements), of 64 / ROW_LANES rows, which are of one tile row. W_hat
// may be W itself (in place): neither is declared restrict.  Bound by memory.  Calls with the host's part, us, a thread per 8 elements with the map in
// device memory -> this: 11008 x 4096, tile 128, f = 1/2 47.0 -> 42.6, 4096 x 4096, tile 64 31.7 -> 26.4, 13824 x 640, tile 128 25.3 -> 20.5; 1048576 x
// 64 69.9 -> 60.7, where a wavefront per row took 153. The matrix passed here starts at the first tile of the map part: `rows` rows and Tk tiles of a
// matrix with K columns.
template <int ROW_LANES>
__global__ __launch_bounds__(256) void apply_mask_kernel(const TileMapArgs map, const uint16_t* W, const uint8_t* __restrict__ mask24, int64_t K, int rows,
                                                         int Tk, int tile_log2, uint16_t* W_hat) {
    constexpr int ROWS = 64 / ROW_LANES, COLS = 8 * ROW_LANES;
    const int cols = Tk << tile_log2, per_row = (cols + COLS - 1) / COLS, units = rows / ROWS * per_row;
    const int lane = threadIdx.x & 63;
    for (int u = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + threadIdx.x / 64)); u < units; u += (int)gridDim.x * 4) {
        const int n = ROWS * (u / per_row), k0 = COLS * (u % per_row), k = k0 + 8 * (lane % ROW_LANES);
        const int t = (n >> tile_log2) * Tk + (k0 >> tile_log2), w = t >> 5, w1 = w + 1 < 2 * kMapGroups ? w + 1 : w;
        const uint64_t bits = (((uint64_t)map.g[w1 >> 1].dense[w1 & 1] << 32) | map.g[w >> 1].dense[w & 1]) >> (t & 31);
        if (k >= cols) continue;
        const int64_t at = (n + lane / ROW_LANES) * K + k;
        union { u32x4 v; uint16_t h[8]; } x;
        x.v = *reinterpret_cast<const u32x4*>(W + at);
        if (!((bits >> ((k - k0) >> tile_log2)) & 1)) {
            union { uint2 v; uint8_t b[8]; } m;
            m.v = *reinterpret_cast<const uint2*>(mask24 + at);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                // M* = M_tile + (1 - M_tile) * M_24 with M_tile = 0 here
                if (!m.b[e]) x.h[e] = 0;
            }
        }
        *reinterpret_cast<u32x4*>(W_hat + at) = x.v;
    }
}

void launch_apply_mask(const uint16_t* W, const uint8_t* mask24, const uint8_t* tile_map, int64_t N, int64_t K, int tile,
                       uint16_t* W_hat, hipStream_t stream) {
    const int64_t Tn = N / tile, Tk = K / tile;
    TileMapArgs map;
    // parts of whole tile rows, or, where a single one is too long, pieces of it
    const int64_t step_k = Tk < kMapTiles ? Tk : kMapTiles, step_n = kMapTiles / step_k;
    for (int64_t tn = 0; tn < Tn; tn += step_n)
        for (int64_t tk = 0; tk < Tk; tk += step_k) {
            const int rn = (int)(Tn - tn < step_n ? Tn - tn : step_n), rk = (int)(Tk - tk < step_k ? Tk - tk : step_k);
            fill_map_args(&map, tile_map + tn * Tk + tk, rn * rk, 0);   // (contiguous: rk = Tk or rn = 1)
            const int64_t at = tn * tile * K + tk * tile, cols = (int64_t)rk * tile;
            const int row_lanes = cols <= 64 ? 8 : cols <= 128 ? 16 : cols <= 256 ? 32 : 64;
            const int64_t units = (int64_t)rn * tile * row_lanes / 64 * ((cols + 511) / 512), blocks = (units + 3) / 4;
            const auto kernel = row_lanes == 8 ? &apply_mask_kernel<8> : row_lanes == 16 ? &apply_mask_kernel<16> : row_lanes == 32 ? &apply_mask_kernel<32>
                                                                                                                              : &apply_mask_kernel<64>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks < 256 * 32 ? blocks : 256 * 32)), dim3(256), 0, stream, map, W + at, mask24 + at, K,
                               rn * tile, rk, tile == 128 ? 7 : 6, W_hat + at);
        }
}

// ------------------------------------------------------------------ hard 2:4 mask from the pattern logits
// Four groups of four consecutive elements per thread and step: the candidate with the largest of the six logits (first one on
// ties; a NaN never wins a comparison), written as four keep bytes.  Candidates in lexicographic order of the kept
// positions: (0,1) (0,2) (0,3) (1,2) (1,3) (2,3).  Bound by memory (24 bytes read, 4 written per group): 11008 x 4096 in 58 us
// (5.4 TB/s); with one group per thread, which is what logits or masks without 16-byte alignment still take, 67 - 73 us.
typedef float pk_f32x4 __attribute__((ext_vector_type(4)));
template <typename F, typename U, int V>
__global__ __launch_bounds__(256) void hard_mask24_kernel(const F* __restrict__ P24, int64_t G, U* __restrict__ mask24) {
    // keep bytes of candidate c, little endian: byte j = element j of the group
    constexpr uint32_t kPattern[6] = {0x00000101u, 0x00010001u, 0x01000001u, 0x00010100u, 0x01000100u, 0x01010000u};
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < G; g += (int64_t)gridDim.x * blockDim.x) {
        F v[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] = __builtin_nontemporal_load(P24 + (int64_t)c * G + g);
        U pat;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            float best = reinterpret_cast<const float*>(&v[0])[e];
            uint32_t p = kPattern[0];
#pragma unroll
            for (int c = 1; c < 6; ++c) {
                const float x = reinterpret_cast<const float*>(&v[c])[e];
                const bool better = x > best;
                best = better ? x : best;
                p = better ? kPattern[c] : p;
            }
            reinterpret_cast<uint32_t*>(&pat)[e] = p;
        }
        mask24[g] = pat;
    }
}

// G is a multiple of 1024 (whole tiles), so the six planes share the alignment of the first.
void launch_hard_mask24(const float* P24, int64_t G, uint8_t* mask24, hipStream_t stream) {
    const bool wide = ((reinterpret_cast<uintptr_t>(P24) | reinterpret_cast<uintptr_t>(mask24)) & 15u) == 0;
    const int64_t n = wide ? G / 4 : G;
    int blocks = (int)((n + 255) / 256);
    if (blocks > 256 * 32) blocks = 256 * 32;
    if (wide)
        hipLaunchKernelGGL((hard_mask24_kernel<pk_f32x4, u32x4, 4>), dim3(blocks), dim3(256), 0, stream, reinterpret_cast<const pk_f32x4*>(P24), n,
                           reinterpret_cast<u32x4*>(mask24));
    else
        hipLaunchKernelGGL((hard_mask24_kernel<float, uint32_t, 1>), dim3(blocks), dim3(256), 0, stream, P24, n, reinterpret_cast<uint32_t*>(mask24));
}

// ------------------------------------------------------------------ compression
__device__ __forceinline__ bool bf16_nonzero(uint16_t h) { return (h & 0x7FFFu) != 0; }

// Compress 4 groups of 4 (16 consecutive elements of one row) into 8 kept values + 16 position bits.
// Returns false if some group holds more than two nonzeros.
__device__ __forceinline__ bool compress16(const uint16_t* in, uint16_t* out, uint32_t& idx) {
    bool ok = true;
    idx = 0;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const uint16_t* grp = in + 4 * g;
        int nnz = 0;
        bool keep[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) { keep[p] = bf16_nonzero(grp[p]); nnz += keep[p] ? 1 : 0; }
        if (nnz > 2) ok = false;
        // fewer than two nonzeros: also keep the lowest-index zeros
#pragma unroll
        for (int p = 0; p < 4; ++p)
            if (!keep[p] && nnz < 2) { keep[p] = true; ++nnz; }
        // first and second kept position and their values, by selects (an element picked by a computed index would go
        // through memory)
        int p0 = 0, p1 = 1, seen = 0;
        uint16_t w0 = grp[0], w1 = grp[1];
#pragma unroll
        for (int p = 0; p < 4; ++p)
            if (keep[p]) {
                if (seen == 0) { p0 = p; w0 = grp[p]; }
                else if (seen == 1) { p1 = p; w1 = grp[p]; }
                ++seen;
            }
        out[2 * g] = w0;
        out[2 * g + 1] = w1;
        idx |= (uint32_t)(p0 | (p1 << 2)) << (4 * g);
    }
    return ok;
}

// One workgroup per tile; every thread requests all its pieces of the tile before it uses the first.  11008 x 4096, tile 128, f = 0.6:
// 33 us (4.8 TB/s) against 41 with a loop over the pieces and kept values picked by a computed index (which the compiler
// sent through LDS); 4096 x 4096, tile 64, f = 0.5: 14 us against 25.
template <int TILE>
__global__ __launch_bounds__(256) void pack_kernel(const TileMapArgs map, int first, const uint16_t* __restrict__ W, int64_t K, int Tk,
                                                   uint8_t* __restrict__ payload, uint32_t* __restrict__ table, uint32_t* __restrict__ slack,
                                                   uint32_t* __restrict__ not_24) {
    constexpr int KPT = TILE / kStepCols, PIECES = TILE * TILE / 8 / 256;
    const int t = first + blockIdx.x;
    const int tn = t / Tk, tk = t % Tk;
    const uint32_t e = map_entry(map, blockIdx.x, t, dense_tile_bytes(TILE), sparse_tile_bytes(TILE));
    if (threadIdx.x == 0) table[t] = e;
    if (t == 0) {
        static_assert(kZeroPad == 256 * sizeof(uint32_t), "one word a thread");
        slack[threadIdx.x] = 0;
    }
    uint8_t* base = payload + entry_offset(e);
    const int lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
    const uint16_t* src = W + ((int64_t)tn * TILE + i) * K + (int64_t)tk * TILE;
    u32x4 in[PIECES];
    if (!entry_sparse(e)) {
#pragma unroll
        for (int p = 0; p < PIECES; ++p) {
            const int f = (threadIdx.x >> 6) + 4 * p, h = f & 1, j = (f >> 1) % KPT, s = (f >> 1) / KPT;   // operand h of fragment (s, j)
            in[p] = *reinterpret_cast<const u32x4*>(src + (int64_t)(16 * s) * K + 64 * j + 32 * h + 8 * q);
        }
#pragma unroll
        for (int p = 0; p < PIECES; ++p) *reinterpret_cast<u32x4*>(base + (size_t)(threadIdx.x + 256 * p) * 16) = in[p];
    } else {
        uint16_t* meta = reinterpret_cast<uint16_t*>(base + sparse_vals_bytes(TILE));
        bool ok = true;
#pragma unroll
        for (int p = 0; p < PIECES / 2; ++p) {
            const int f = (threadIdx.x >> 6) + 4 * p, j = f % KPT, s = f / KPT;
            const u32x4* at = reinterpret_cast<const u32x4*>(src + (int64_t)(16 * s) * K + 64 * j + 16 * q);
            in[2 * p] = at[0];
            in[2 * p + 1] = at[1];
        }
#pragma unroll
        for (int p = 0; p < PIECES / 2; ++p) {
            const int f = (threadIdx.x >> 6) + 4 * p, j = f % KPT, s = f / KPT;
            union { u32x4 v[2]; uint16_t h[16]; } x;
            x.v[0] = in[2 * p];
            x.v[1] = in[2 * p + 1];
            union { u32x4 v; uint16_t h[8]; } out;
            uint32_t idx;
            ok = compress16(x.h, out.h, idx) && ok;
            *reinterpret_cast<u32x4*>(base + (size_t)(threadIdx.x + 256 * p) * 16) = out.v;
            meta[(s * 64 + lane) * KPT + j] = (uint16_t)idx;
        }
        if (!ok) report_not_24(not_24);
    }
}

void launch_pack(const uint16_t* W, int64_t K, const uint8_t* tile_map, int n_tiles, int Tk, int tile, uint8_t* payload, uint32_t* d_table,
                 uint32_t* slack, uint32_t* not_24, hipStream_t stream) {
    TileMapArgs map;
    uint32_t before = 0;
    for (int first = 0; first < n_tiles; first += kMapTiles) {
        const int n = n_tiles - first < kMapTiles ? n_tiles - first : kMapTiles;
        before = fill_map_args(&map, tile_map + first, n, before);
        hipLaunchKernelGGL(tile == 128 ? &pack_kernel<128> : &pack_kernel<64>, dim3(n), dim3(256), 0, stream, map, first, W, K, Tk, payload, d_table, slack, not_24);
    }
}

// ------------------------------------------------------------------ decompression
__global__ __launch_bounds__(256) void unpack_kernel(const uint8_t* __restrict__ payload, const uint32_t* __restrict__ table, int Tk,
                                                     int tile, int64_t K, uint16_t* __restrict__ W_out) {
    const int t = blockIdx.x;
    const int tn = t / Tk, tk = t % Tk;
    const uint32_t e = table[t];
    const uint8_t* base = payload + entry_offset(e);
    const int64_t n0 = (int64_t)tn * tile, k0 = (int64_t)tk * tile;
    const int KPT = tile / kStepCols;
    if (!entry_sparse(e)) {
        const int nchunks = tile * tile / 8;
        for (int c = threadIdx.x; c < nchunks; c += blockDim.x) {
            const int lane = c & 63, h = (c >> 6) & 1, sj = c >> 7;
            const int j = sj % KPT, s = sj / KPT, i = lane & 15, q = lane >> 4;
            uint16_t* dst = W_out + (n0 + 16 * s + i) * K + k0 + 64 * j + 32 * h + 8 * q;
            *reinterpret_cast<u32x4*>(dst) = *reinterpret_cast<const u32x4*>(base + (size_t)c * 16);
        }
    } else {
        const int nchunks = tile * tile / 16;
        const uint16_t* meta = reinterpret_cast<const uint16_t*>(base + sparse_vals_bytes(tile));
        for (int c = threadIdx.x; c < nchunks; c += blockDim.x) {
            const int lane = c & 63, sj = c >> 6;
            const int j = sj % KPT, s = sj / KPT, i = lane & 15, qa = lane >> 4;
            union { u32x4 v; uint16_t h[8]; } in;
            in.v = *reinterpret_cast<const u32x4*>(base + (size_t)c * 16);
            const uint32_t idx = meta[(s * 64 + lane) * KPT + j];
            union { u32x4 v[2]; uint16_t h[16]; } out;
            out.v[0] = u32x4{0, 0, 0, 0};
            out.v[1] = u32x4{0, 0, 0, 0};
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int p0 = (idx >> (4 * g)) & 3, p1 = (idx >> (4 * g + 2)) & 3;
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    uint16_t v = 0;
                    if (p == p0) v = in.h[2 * g];
                    if (p == p1) v = in.h[2 * g + 1];
                    out.h[4 * g + p] = v;
                }
            }
            uint16_t* dst = W_out + (n0 + 16 * s + i) * K + k0 + 64 * j + 16 * qa;
            *reinterpret_cast<u32x4*>(dst) = out.v[0];
            *reinterpret_cast<u32x4*>(dst + 8) = out.v[1];
        }
    }
}

void launch_unpack(const uint8_t* payload, const uint32_t* d_table, int n_tiles, int Tk, int tile, int64_t K, uint16_t* W_out,
                   hipStream_t stream) {
    hipLaunchKernelGGL(unpack_kernel, dim3(n_tiles), dim3(256), 0, stream, payload, d_table, Tk, tile, K, W_out);
}

}  // namespace patch
