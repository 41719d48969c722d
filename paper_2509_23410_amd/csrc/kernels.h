// Internal launch interface between the C ABI (api.hip) and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// records the hipError_t that patch_last_hip_error reports (thread-local, in api.hip)
void patch_note_hip_error(int hip_error);

namespace patch {

// A part of a tile map as kernel arguments (4096 bytes at most, the hidden ones included), so that no launch has to wait for a copy of the map: 64
// tiles a group, bit set = dense, and how many of the whole map's tiles before the group are.
constexpr int kMapGroups = 304, kMapTiles = 64 * kMapGroups;
struct TileMapArgs {
    struct { uint32_t dense[2], before; } g[kMapGroups];
};
// `before` = dense tiles in front of map[0]; returns those in front of map[n]
uint32_t fill_map_args(TileMapArgs* a, const uint8_t* map, int n, uint32_t before);

// tile_map on the host; launches as many kernels as its tiles need
void launch_apply_mask(const uint16_t* W, const uint8_t* mask24, const uint8_t* tile_map, int64_t N, int64_t K, int tile,
                       uint16_t* W_hat, hipStream_t stream);
// mask24 (N x K keep bytes, 4-byte aligned) from the 6 x G pattern logits, G = N K / 4 groups
void launch_hard_mask24(const float* P24, int64_t G, uint8_t* mask24, hipStream_t stream);
// tile_map on the host; also writes d_table (an entry per tile) and zeroes the kZeroPad bytes at `slack`.  *not_24 (device view of host memory) is set
// to 1 if a group of four of a 2:4 tile holds more than two nonzeros.
void launch_pack(const uint16_t* W, int64_t K, const uint8_t* tile_map, int n_tiles, int Tk, int tile, uint8_t* payload, uint32_t* d_table,
                 uint32_t* slack, uint32_t* not_24, hipStream_t stream);
// n words (any number) to dst by kernel arguments
void launch_put_words(uint32_t* dst, const uint32_t* src, size_t n, hipStream_t stream);
void launch_unpack(const uint8_t* payload, const uint32_t* d_table, int n_tiles, int Tk, int tile, int64_t K, uint16_t* W_out,
                   hipStream_t stream);

// Operands shared by the GEMM launchers.
struct GemmArgs {
    const uint16_t* X;   // M x K bf16
    int64_t M, N, K;
    int tile, Tn, Tk;
    const uint8_t* payload;
    const uint32_t* table;  // Tn x Tk entries
    float* Y;               // M x N fp32
    float* ws = nullptr;    // caller's workspace for split-K partial products (prefill), may be null
    size_t ws_bytes = 0;
    int n_cus;
    int ybf16 = 0;          // nonzero: Y (and every Y of a set) is bf16, the accumulator rounded to nearest even
    int sparse_pct = 0;     // share of 2:4 tiles in the weight (all weights of a set), per cent: a hint for schedules
};

// Up to kMaxMany weights that share one X (same K, same tile), multiplied in one launch.  The launch numbers its
// units of features (decode: 16-feature strips; prefill: 256-feature blocks, each weight rounded up) across all
// weights; first[i] is the first unit of weight i.
constexpr int kMaxMany = 8;
struct WeightSet {
    const uint8_t* payload[kMaxMany];
    const uint32_t* table[kMaxMany];
    float* Y[kMaxMany];          // M x N[i] fp32
    int64_t N[kMaxMany];
    int first[kMaxMany];
    int count, units;            // weights, units in total
};
typedef WeightSet DecodeSet;
// A set of one, for the kernels' single-weight instantiations: 32 bytes of kernel arguments instead of 300.  Every
// wavefront reads its arguments before it can request anything else, the set's arrays in several dependent rounds
// (which weight? then that weight's pointers), and a decode launch is short enough for that to show.
struct WeightOne {
    const uint8_t* payload;
    const uint32_t* table;
    float* Y;
    int64_t N;
};

constexpr int kDecodeRows = 64;    // rows of X per decode launch
constexpr int kBatchRows = 128;    // batch_kernel
// The rows of a strip-kernel or mid_kernel pass may be dealt over up to `deal` workgroups per feature group (gridDim.z; 1, 2 or 4), whole blocks of 16 each: the rows of one,
// and how many workgroups that makes
inline int rows_each(int rows, int deal) { return deal > 1 ? 16 * (((rows + 15) / 16 + deal - 1) / deal) : rows; }
inline unsigned rows_deals(int rows, int each) { return (unsigned)((rows + each - 1) / each); }
// gridDim.x of a launch over `units` feature groups (K whole) whose rows are dealt: a multiple of 8, workgroups beyond `units` end at once.  Workgroups go to the eight dies in
// turn by their linear index, each die with an L2 of its own: those that share a feature group's weights then meet in one L2, and memory sends the weights
// once.  64 rows, units as they are -> rounded up: three 896 x 896 (42 groups) 5.3 -> 5.1 us, weights cold 7.1 -> 5.9; 40 rows of 4864 x 13824, f = 1/2 (76) 47.5 -> 39.7;
// 24 rows of 5504 x 2048, f = 0 (86) 12.0 -> 9.4.  Not where the fullest die would need one more round of its compute units than all of them together, nor for
// K in chunks (896 x 4864 in 6 chunks, 3 deals: 36 workgroups on the 32 units of a die, 7.4 -> 10.1; in 8 and 2, no round more, 2 % slower: few bytes a group).
inline unsigned deal_units(int units, unsigned deals, int n_cus) {
    const int each = (int)deals, die = n_cus / 8, up = (units + 7) / 8;
    return (unsigned)(deals > 1 && (up * each + die - 1) / die <= (units * each + n_cus - 1) / n_cus ? 8 * up : units);
}

// Up to kDecodeRows rows of X starting at row m0 (decode shape; 16-row blocks, the weights streamed once per launch).
// split_k = K slices (wavefronts) per workgroup, 0 picks a default.  Returns the number used.
int launch_decode(const GemmArgs& a, int64_t m0, int rows, int split_k, int variant, hipStream_t stream, int deal = 1);
// The same for a set of weights; a supplies X, K, tile, Tk, n_cus (its payload / table / Y / N are ignored).
int launch_decode_set(const GemmArgs& a, const DecodeSet& set, int64_t m0, int rows, int split_k, int variant, hipStream_t stream, int deal = 1);

// Up to kDecodeRows rows of X starting at row m0 (batched decode): 64 features per wavefront, so X is read once per
// four strips.  set.units / first[] count 64-feature groups.  split > 1 (single weight only, a.ws must hold
// split x rows x N floats) cuts K into chunks over more workgroups; mid_split picks the count (1 without a.ws).
int mid_split(const GemmArgs& a, int rows, int requested, int deals = 1);
void launch_mid_set(const GemmArgs& a, const WeightSet& set, int64_t m0, int rows, int split, hipStream_t stream, int deal = 1);
// Y[i] = sum over the slices of ws[slice * n4 + i] (float4 units), slice 0 first
void wr_reduce(const float* ws, size_t n4, int slices, float* Y, int ybf16, hipStream_t stream);

// the same for a set: the slices of weight i, n4[i] float4 each, one behind the other at ws[i]
struct WrReduceSet {
    const float* ws[kMaxMany];
    float* Y[kMaxMany];
    size_t n4[kMaxMany];
};
void wr_reduce_set(const WrReduceSet& red, int count, int slices, int ybf16, hipStream_t stream);
// Up to kBatchRows rows of X starting at row m0: 128 features per workgroup.  set.units / first[] count groups of 128
// features, each weight rounded up; split > 1 needs a.ws with room for split x rows x N floats of every weight.
void launch_batch_set(const GemmArgs& a, const WeightSet& set, int64_t m0, int rows, int split, hipStream_t stream);

// Any M (prefill shape).
void launch_prefill(const GemmArgs& a, int variant, int split_k, hipStream_t stream);
bool prefill_wreg_supports(const GemmArgs& a);                  // K <= 16384, M * K * 2 < 4 GB
int prefill_wreg_split(const GemmArgs& a, int requested);       // K slices per output tile the launch will use
int prefill_lds_split(const GemmArgs& a, int requested, int bm = 256);   // the same for the LDS-staged kernel with blocks of bm rows
// whether the default choice (variant 0, no split requested) is prefill_kernel_areg with blocks of 128 rows, and its split, where prefill_r128_split does
// not take the launch; no_w64: see there
bool prefill_prefers_128_rows(const GemmArgs& a, int* split, bool no_w64 = false);
double prefill_estimate(const GemmArgs& a);                                       // us the default choice is estimated to take at few rows
double prefill_set_estimate(const GemmArgs& a, const int64_t* N, int count);      // the same for a set of weights of N[i] features
double pf_few_rows(const GemmArgs& a, int64_t N, int blocks, int split, bool rows128, bool whole_blocks);   // what both go by
// How an unsplit launch of 256 x 256 tiles runs its part-filled last round: the last `tail` tiles (0: as the others) in `slices` K slices (more than one
// needs a.ws with a slot of 256 x 256 floats per tile and slice), by prefill_kernel_r128 (`halves`: 128 rows a workgroup) or by the kernel of the rest.
struct LastRound { int tail, slices; bool halves; };
LastRound prefill_wreg_tail(const GemmArgs& a);
size_t prefill_wreg_tail_bytes(const GemmArgs& a);   // see there
LastRound prefill_wreg_last_round(int tiles, const GemmArgs& a);   // the same for a given tile count (sets of weights)
void launch_prefill_wreg_rounds(const GemmArgs& a, const WeightSet& set, int tiles_m, const LastRound& r, hipStream_t stream);
// Price of a prefill launch in us (prefill_r128_split has the formula and what it was fitted to)
struct PrefillPrice { double base, begin, t0, t1, g1, g2, second, rate; };
constexpr PrefillPrice kPriceR128 = {6.7, 2.3, 0.682, 0.171, 0.365, 0.0, 2.2, 10.3e6}, kPriceAreg128 = {4.6, 3.2, 0.864, 0.199, 0.347, 0.0, 3.3, 13.0e6},
                       kPriceWreg = {10.6, 0.5, 0.841, 0.411, 0.017, 0.364, 1.6, 8.4e6};
double pf_price(const PrefillPrice& p, const GemmArgs& a, int64_t N, int64_t blocks, int split);
void launch_prefill_wreg(const GemmArgs& a, int split_k, hipStream_t stream);
// The same for a set of weights; a supplies X, M, K, tile, Tk, n_cus and, optionally, ws / ws_bytes (then a
// part-filled last round is split as in launch_prefill_wreg).  All of the set must pass prefill_wreg_supports with
// these M, K.
void launch_prefill_wreg_set(const GemmArgs& a, const WeightSet& set, hipStream_t stream);
int prefill_wreg_set_split(const GemmArgs& a, int blocks, int64_t N);   // K slices of such a launch over `blocks` output tiles, N features in all
// Blocks of 256 features x 128 rows by wavefronts of 64 features; a, set as above; split > 1 needs a.ws with room for split x M x N floats of every
// weight.  prefill_r128_split: the K slices in which the default choice (variant 0, no split requested) runs `count` weights of N[i] features this
// way, 0 = it does not.
int prefill_r128_split(const GemmArgs& a, const int64_t* N, int count);
void launch_prefill_r128(const GemmArgs& a, const WeightSet& set, int split, hipStream_t stream);
// Tiles t0 .. t0 + tail - 1 of a launch over 256 x 256 tiles, two workgroups each; slices > 1: partial tiles to slots of 256 x 256 floats at set.Y
void launch_prefill_r128_tail(const GemmArgs& a, const WeightSet& set, int tiles_m, int t0, int tail, int slices, hipStream_t stream);

}  // namespace patch

// Test hooks: exported like the interface in patch.h, but no part of it.
struct patch_packed;
struct patch_packed4;
extern "C" {
// The prefill product of `count` weights sharing X by prefill_kernel_r128 in `split` K slices, whatever the dispatch would take.
int patch_test_prefill128(const void* X, int64_t M, const patch_packed* const* P, void* const* Y, int count, int split, int y_bf16, void* workspace,
                          size_t workspace_bytes, void* stream);
// What AUTO takes for M rows of `count` weights of N[i] x K features sharing X (sparse_pct per cent of the tiles 2:4) given ws_bytes of
// workspace on 256 compute units: kernel (0 strip, 1 mid, 2 batch, 3 the prefill path, 4 that in blocks of 128 rows by
// prefill_prefers_128_rows) and K chunks of every pass (1 for kernel 3), at most 8; returns their number, -1 = bad arguments.  Runs on the host alone.
int patch_test_schedule(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes, int* kernel, int* chunks);
// The same and, per pass, over how many workgroups per feature group its rows are dealt (rows_deals; 1 = not).
int patch_test_schedule_deals(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes, int* kernel, int* chunks, int* deals);
// The prefill product of `count` weights by the 256-row register-weight kernel, its last round (the tiles beyond a multiple of the compute units) in
// `slices` K slices, `halves` as in LastRound; halves = -1: as the rest of the launch.
int patch_test_prefill_last_round(const void* X, int64_t M, const patch_packed* const* P, void* const* Y, int count, int halves, int slices, int y_bf16,
                                  void* workspace, size_t workspace_bytes, void* stream);
// prefill_wreg_last_round for such a launch (arguments as in patch_test_schedule): returns its tail, -1 = bad arguments
int patch_test_last_round(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes, int* slices, int* halves);
// prefill_r128_split of the same, for the prefill path
int patch_test_prefill128_split(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes);
// fill_map_args of n <= 19456 tiles, `before` dense ones in front of them: three words per 64 tiles to out; returns the dense tiles up to the end, -1 = bad arguments
int64_t patch_test_map_args(const uint8_t* map, int n, uint32_t before, uint32_t* out);
// deal_units: gridDim.x of a launch over `units` feature groups whose rows go over `deals` workgroups
int patch_test_deal_units(int units, int deals, int n_cus);
// The 4-bit product of `count` weights sharing X by one kernel, whatever the dispatch would take: 0 the strip kernel, 1 batch4_kernel, both in
// passes of up to 64 rows, 2 / 3 the prefill-shaped kernel in blocks of 128 / 256 rows, 4 the one with two K groups, 5 the same with the blocks
// beyond a multiple of the compute units in `chunks` K slices (slots of 128 KB).  2 - 5: a single weight.  chunks > 1 (a single weight,
// kernels 1 - 4): K in that many chunks over the workspace.
int patch_test_gemm4(const void* X, int64_t M, const patch_packed4* const* P, void* const* Y, int count, int kernel, int chunks,
                     void* workspace, size_t workspace_bytes, void* stream);
// patch_test_schedule for patch_gemm4_ex (count 1) and patch_gemm4_many: kernels as in patch_test_gemm4.
int patch_test_schedule4(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes, int* kernel, int* chunks);
// Adds to the uint32 at `mismatches` (device) how often the conversion of bf16 outputs differs from rounding on the bit pattern, over all 2^32 patterns.
int patch_test_bf16_mismatches(void* mismatches, void* stream);
}
