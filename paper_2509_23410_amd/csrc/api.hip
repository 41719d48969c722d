// C ABI of the library (see include/patch.h): argument checks, the patch_packed object, host-side table
// construction and kernel dispatch.  No device arithmetic here.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <new>
#include <tuple>
#include <vector>

#include "../../include/patch.h"
#include "host_word.h"
#include "kernels.h"
#include "layout.h"
#include "saved.h"

using namespace patch;

struct patch_packed {
    int64_t N = 0, K = 0;
    int tile = 0;
    int Tn = 0, Tk = 0;
    int64_t n_sparse = 0;
    size_t payload_bytes = 0;   // sum of tile payloads (no alignment slack: tiles are granule multiples)
    // one allocation: payload | zeroed slack | table | pairs
    uint8_t* d_payload = nullptr;
    uint32_t* d_table = nullptr;
    std::vector<uint8_t> tile_map;   // host copy, 1 = dense
    std::vector<uint32_t> table;     // host copy of the offset / type table
    std::vector<int32_t> pairs;      // tile rows two by two (see pair_tile_rows); behind the table on the device
    int device = 0;
    int n_cus = 256;
};

static thread_local int g_last_hip_error = 0;
void patch_note_hip_error(int hip_error) { g_last_hip_error = hip_error; }

#define HIP_TRY(expr)                                   \
    do {                                                \
        hipError_t e_ = (expr);                         \
        if (e_ != hipSuccess) {                         \
            g_last_hip_error = (int)e_;                 \
            return PATCH_ERR_HIP;                       \
        }                                               \
    } while (0)

static patch_status check_shape(int64_t N, int64_t K, int tile) {
    if (N <= 0 || K <= 0) return PATCH_ERR_ARG;
    if (tile != 64 && tile != 128) return PATCH_ERR_SHAPE;
    if (N % tile != 0 || K % tile != 0) return PATCH_ERR_SHAPE;
    if (N / tile > (1 << 20) || K / tile > (1 << 20)) return PATCH_ERR_SHAPE;
    return PATCH_OK;
}

// Which two tile rows share a prefill workgroup (tile-map-driven schedule; the paper leaves the schedule to the
// implementation).  The workgroup's wavefronts meet at a barrier every 64-column step, so a step in which one tile row
// is dense and the other 2:4 lasts as long as a dense one: a pair costs about Tk - 0.3 x (steps in which BOTH rows
// are 2:4).  Rows are therefore paired so that these common 2:4 steps are many: within windows of 256 rows, the free
// pair with the most of them first (ties: lowest row indices; counting agreeing steps of either type instead
// measured 1 - 3 % slower).  Returns 2 * ceil(Tn / 2) entries, pair p = rows out[2 p], out[2 p + 1]; -1 = no
// second row.
static std::vector<int32_t> pair_tile_rows(const std::vector<uint8_t>& tile_map, int Tn, int Tk) {
    std::vector<int32_t> out;
    out.reserve((size_t)Tn + 1);
    std::vector<int> carry;  // rows left single by earlier windows
    constexpr int kWindow = 256;
    // the 2:4 tiles of a row as a bit set (86 rows of 32 tiles, 3655 pairs: 40 us, byte by byte and with a comparison sort 300)
    const int words = (Tk + 63) / 64;
    std::vector<uint64_t> bits((size_t)Tn * words, 0);
    for (int r = 0; r < Tn; ++r)
        for (int k = 0; k < Tk; ++k) bits[(size_t)r * words + k / 64] |= (uint64_t)(tile_map[(size_t)r * Tk + k] == 0) << (k % 64);
    const auto common = [&](int a, int b) {   // steps in which both rows are 2:4
        int n = 0;
        for (int i = 0; i < words; ++i) n += __builtin_popcountll(bits[(size_t)a * words + i] & bits[(size_t)b * words + i]);
        return n;
    };
    std::vector<uint32_t> cand, sorted;   // pairs of positions in the window, i << 16 | j
    std::vector<int> agree, first((size_t)Tk + 2);
    for (int w0 = 0; w0 < Tn; w0 += kWindow) {
        std::vector<int> rows = carry;
        carry.clear();
        for (int r = w0; r < Tn && r < w0 + kWindow; ++r) rows.push_back(r);
        const int n = (int)rows.size();
        cand.clear();
        agree.clear();
        std::fill(first.begin(), first.end(), 0);
        for (int i = 0; i < n; ++i)
            for (int j = i + 1; j < n; ++j) {
                const int c = common(rows[i], rows[j]);
                cand.push_back((uint32_t)i << 16 | (uint32_t)j);
                agree.push_back(c);
                ++first[Tk - c + 1];
            }
        // most common steps first, pairs of equal count in their order (a counting sort)
        for (int c = 0; c <= Tk; ++c) first[c + 1] += first[c];
        sorted.resize(cand.size());
        for (size_t p = 0; p < cand.size(); ++p) sorted[first[Tk - agree[p]]++] = cand[p];
        std::vector<char> used((size_t)n, 0);
        int left = n;
        for (size_t p = 0; p < sorted.size() && left > 1; ++p) {
            const int a = (int)(sorted[p] >> 16), b = (int)(sorted[p] & 0xFFFFu);
            if (used[a] || used[b]) continue;
            used[a] = used[b] = 1;
            left -= 2;
            out.push_back(rows[a]);
            out.push_back(rows[b]);
        }
        for (int i = 0; i < n; ++i)
            if (!used[i]) carry.push_back(rows[i]);
    }
    for (size_t i = 0; i + 1 < carry.size(); i += 2) { out.push_back(carry[i]); out.push_back(carry[i + 1]); }
    if (carry.size() % 2) { out.push_back(carry.back()); out.push_back(-1); }
    // Order of the pairs = order of the feature blocks in the launch, of which every XCD runs a contiguous piece
    // (all, a half or a quarter of it, depending on M), its workgroups starting in that order as compute units
    // become free.  A pair costs about Tk - 0.3 x (steps in which both rows are 2:4).  The pairs are dealt by falling
    // cost into four piles, laid one after the other: every quarter of the order carries about the average cost, and
    // inside it the heaviest workgroups start first (alternating heaviest / lightest measured 0 - 4 % slower).
    const size_t np = out.size() / 2;
    std::vector<std::pair<int, size_t>> cost(np);
    for (size_t p = 0; p < np; ++p) {
        const int a = out[2 * p], b2 = out[2 * p + 1];
        cost[p] = {common(a, b2 < 0 ? a : b2), p};  // more common 2:4 steps = lighter
    }
    std::stable_sort(cost.begin(), cost.end(), [](const auto& x, const auto& y) { return x.first < y.first; });
    std::vector<int32_t> ordered;
    ordered.reserve(out.size());
    constexpr size_t kPiles = 4;
    for (size_t pile = 0; pile < kPiles; ++pile)
        for (size_t r = pile; r < np; r += kPiles) {
            const size_t h = cost[r].second;
            ordered.push_back(out[2 * h]); ordered.push_back(out[2 * h + 1]);
        }
    return ordered;
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Library-side scratch for patch_gemm_static (callers that cannot allocate): split-K partial products live here
// instead of a caller workspace.  One copy per GPU, held until the process ends.  In host code the array's name is
// only a handle for hipGetSymbolAddress; the device address is looked up once per device and kept.
constexpr size_t kStaticScratchBytes = PATCH_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call per device).
static patch_status static_scratch(void** out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return PATCH_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) { g_last_hip_error = (int)hipErrorInvalidSymbol; return PATCH_ERR_HIP; }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return PATCH_OK;
}

extern "C" {

const char* patch_version(void) { return "patch-mi355x 0.1 (gfx950)"; }

int patch_last_hip_error(void) { return g_last_hip_error; }

const char* patch_strerror(patch_status s) {
    switch (s) {
        case PATCH_OK: return "ok";
        case PATCH_ERR_ARG: return "invalid argument (null or misaligned pointer, non-positive size, unknown option)";
        case PATCH_ERR_SHAPE: return "unsupported shape (tile must be 64 or 128 and divide N and K)";
        case PATCH_ERR_NOT_24: return "a group of four in a 2:4 tile holds more than two nonzeros";
        case PATCH_ERR_ALLOC: return "allocation failed";
        case PATCH_ERR_HIP: return "HIP runtime error";
        case PATCH_ERR_SIZE: return "caller buffer too small";
        case PATCH_ERR_NOT_FOUND: return "no tuned schedule stored for this key";
    }
    return "unknown status";
}

patch_status patch_apply_mask(const void* W, const void* mask24, const uint8_t* tile_map, int64_t N, int64_t K, int tile,
                              void* W_hat, void* stream) {
    if (!W || !mask24 || !tile_map || !W_hat) return PATCH_ERR_ARG;
    patch_status st = check_shape(N, K, tile);
    if (st != PATCH_OK) return st;
    if (!aligned16(W) || !aligned16(W_hat) || (reinterpret_cast<uintptr_t>(mask24) & 7u)) return PATCH_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    launch_apply_mask(static_cast<const uint16_t*>(W), static_cast<const uint8_t*>(mask24), tile_map, N, K, tile, static_cast<uint16_t*>(W_hat), s);
    hipError_t e = hipGetLastError();
    const hipError_t e_sync = hipStreamSynchronize(s);
    if (e == hipSuccess) e = e_sync;
    if (e != hipSuccess) { g_last_hip_error = (int)e; return PATCH_ERR_HIP; }
    return PATCH_OK;
}

patch_status patch_hard_masks(const float* P_tile, const void* P_24, int64_t N, int64_t K, int tile, uint8_t* tile_map,
                              void* mask24, void* stream) {
    if (!P_tile || !P_24 || !tile_map || !mask24) return PATCH_ERR_ARG;
    patch_status st = check_shape(N, K, tile);
    if (st != PATCH_OK) return st;
    if ((reinterpret_cast<uintptr_t>(P_24) & 3u) || (reinterpret_cast<uintptr_t>(mask24) & 7u)) return PATCH_ERR_ARG;
    const size_t T = (size_t)(N / tile) * (size_t)(K / tile);
    for (size_t i = 0; i < T; ++i) tile_map[i] = (P_tile[i] > 0.0f) ? 1 : 0;   // NaN and 0: the 2:4 class
    launch_hard_mask24(static_cast<const float*>(P_24), N * K / 4, static_cast<uint8_t*>(mask24), static_cast<hipStream_t>(stream));
    HIP_TRY(hipGetLastError());
    return PATCH_OK;
}

void patch_free(patch_packed* P) {
    if (!P) return;
    if (P->d_payload) (void)hipFree(P->d_payload);
    delete P;
}

// The host side of a packed weight (tile map, offset / type table) and its device buffers, one allocation; nothing of it written yet: patch_pack's kernel
// writes payload, slack and table, patch_deserialize copies them.
static patch_status new_packed(int64_t N, int64_t K, const uint8_t* tile_map, int tile, patch_packed** out) {
    patch_packed* P = new (std::nothrow) patch_packed();
    if (!P) return PATCH_ERR_ALLOC;
    P->N = N; P->K = K; P->tile = tile;
    P->Tn = (int)(N / tile); P->Tk = (int)(K / tile);
    const size_t T = (size_t)P->Tn * (size_t)P->Tk;
    try {
        P->tile_map.resize(T);
        P->table.resize(T);
    } catch (...) { delete P; return PATCH_ERR_ALLOC; }
    uint64_t off = 0;
    for (size_t i = 0; i < T; ++i) {
        const bool sparse = tile_map[i] == 0;
        P->tile_map[i] = sparse ? 0 : 1;
        P->table[i] = make_entry(off, sparse);
        off += sparse ? sparse_tile_bytes(tile) : dense_tile_bytes(tile);
        if (sparse) ++P->n_sparse;
    }
    P->payload_bytes = off;
    if ((off / kGranule) >> 31) { delete P; return PATCH_ERR_SHAPE; }

    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
        g_last_hip_error = (int)hipGetLastError();
        delete P;
        return PATCH_ERR_HIP;
    }
    P->device = dev;
    P->n_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;

    const size_t n_pairs = tile == 128 ? 2 * (((size_t)P->Tn + 1) / 2) : 0;
    // (a kilobyte of zeroed slack behind the payload keeps any over-read of the last tile inside the allocation)
    if (hipMalloc(&P->d_payload, P->payload_bytes + kZeroPad + (T + n_pairs) * sizeof(uint32_t)) != hipSuccess) {
        (void)hipGetLastError();
        patch_free(P);
        return PATCH_ERR_ALLOC;
    }
    P->d_table = reinterpret_cast<uint32_t*>(P->d_payload + P->payload_bytes + kZeroPad);
    *out = P;
    return PATCH_OK;
}

// The tile-row pairs of a new packed weight, uploaded on `s` (tile 128 only: prefill_kernel_wreg reads them).
static patch_status add_pairs(patch_packed* P, hipStream_t s) {
    if (P->tile != 128) return PATCH_OK;
    try {
        P->pairs = pair_tile_rows(P->tile_map, P->Tn, P->Tk);
    } catch (...) { return PATCH_ERR_ALLOC; }
    launch_put_words(P->d_table + P->table.size(), reinterpret_cast<const uint32_t*>(P->pairs.data()), P->pairs.size(), s);
    HIP_TRY(hipGetLastError());
    return PATCH_OK;
}

patch_status patch_pack(const void* W_hat, int64_t N, int64_t K, const uint8_t* tile_map, int tile, void* stream,
                        patch_packed** out) {
    if (!W_hat || !tile_map || !out) return PATCH_ERR_ARG;
    patch_status st = check_shape(N, K, tile);
    if (st != PATCH_OK) return st;
    if (!aligned16(W_hat)) return PATCH_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HostWord not_24;
    if (!not_24.valid()) return PATCH_ERR_ALLOC;
    patch_packed* P = nullptr;
    st = new_packed(N, K, tile_map, tile, &P);
    if (st != PATCH_OK) return st;
    launch_pack(static_cast<const uint16_t*>(W_hat), K, P->tile_map.data(), (int)P->table.size(), P->Tk, tile, P->d_payload, P->d_table,
                reinterpret_cast<uint32_t*>(P->d_payload + P->payload_bytes), not_24.device(), s);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) st = add_pairs(P, s);   // on the host while the kernel runs
    const hipError_t e_sync = hipStreamSynchronize(s);
    if (e == hipSuccess) e = e_sync;
    if (e != hipSuccess && st == PATCH_OK) { g_last_hip_error = (int)e; st = PATCH_ERR_HIP; }
    if (st == PATCH_OK && not_24.value()) st = PATCH_ERR_NOT_24;
    if (st != PATCH_OK) {
        patch_free(P);
        return st;
    }
    *out = P;
    return PATCH_OK;
}

// ---- a packed weight saved to and loaded from host memory (saved.h)
size_t patch_serialized_bytes(const patch_packed* P) {
    if (!P) return 0;
    return saved_round(sizeof(SavedHeader)) + saved_round(P->tile_map.size()) + P->payload_bytes;
}

patch_status patch_serialize(const patch_packed* P, void* buf, size_t bytes, void* stream) {
    if (!P || !buf) return PATCH_ERR_ARG;
    if (bytes < patch_serialized_bytes(P)) return PATCH_ERR_SIZE;
    uint8_t* b = static_cast<uint8_t*>(buf);
    const size_t map_at = saved_round(sizeof(SavedHeader)), pay_at = map_at + saved_round(P->tile_map.size());
    memset(b, 0, pay_at);
    memcpy(b + map_at, P->tile_map.data(), P->tile_map.size());
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIP_TRY(hipMemcpyAsync(b + pay_at, P->d_payload, P->payload_bytes, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    SavedHeader h = {};
    memcpy(h.magic, kSavedMagic16, 8);
    h.layout = kSavedLayout;
    h.tile = (uint32_t)P->tile;
    h.N = P->N;
    h.K = P->K;
    h.map_bytes = P->tile_map.size();
    h.payload_bytes = P->payload_bytes;
    h.checksum = fnv1a(b + pay_at, P->payload_bytes, fnv1a(b + map_at, P->tile_map.size(), kFnvBasis));
    memcpy(b, &h, sizeof(h));
    return PATCH_OK;
}

patch_status patch_deserialize(const void* buf, size_t bytes, void* stream, patch_packed** out) {
    if (!buf || !out) return PATCH_ERR_ARG;
    if (bytes < saved_round(sizeof(SavedHeader))) return PATCH_ERR_SIZE;
    const uint8_t* b = static_cast<const uint8_t*>(buf);
    SavedHeader h;
    memcpy(&h, b, sizeof(h));
    if (memcmp(h.magic, kSavedMagic16, 8) != 0 || h.layout != kSavedLayout) return PATCH_ERR_ARG;
    const patch_status shape = check_shape(h.N, h.K, (int)h.tile);
    if (shape != PATCH_OK) return shape;
    const uint64_t T = (uint64_t)(h.N / h.tile) * (uint64_t)(h.K / h.tile);
    if (h.map_bytes != T || h.aux_bytes != 0) return PATCH_ERR_ARG;
    const size_t map_at = saved_round(sizeof(SavedHeader)), pay_at = map_at + saved_round((size_t)T);
    if (bytes < pay_at || h.payload_bytes > bytes - pay_at) return PATCH_ERR_SIZE;
    for (uint64_t i = 0; i < T; ++i)
        if (b[map_at + i] > 1) return PATCH_ERR_ARG;
    if (fnv1a(b + pay_at, (size_t)h.payload_bytes, fnv1a(b + map_at, (size_t)T, kFnvBasis)) != h.checksum) return PATCH_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    patch_packed* P = nullptr;
    patch_status st = new_packed(h.N, h.K, b + map_at, (int)h.tile, &P);
    if (st != PATCH_OK) return st;
    if (P->payload_bytes != h.payload_bytes) {   // the map decides the size: a header that disagrees is not ours
        patch_free(P);
        return PATCH_ERR_ARG;
    }
    constexpr uint32_t kZeroes[kZeroPad / sizeof(uint32_t)] = {};
    launch_put_words(reinterpret_cast<uint32_t*>(P->d_payload + P->payload_bytes), kZeroes, kZeroPad / sizeof(uint32_t), s);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(P->d_table, P->table.data(), P->table.size() * sizeof(uint32_t), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(P->d_payload, b + pay_at, P->payload_bytes, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) st = add_pairs(P, s);
    const hipError_t e_sync = hipStreamSynchronize(s);   // the caller's buffer is free to go when the call returns
    if (e == hipSuccess) e = e_sync;
    if (e != hipSuccess && st == PATCH_OK) { g_last_hip_error = (int)e; st = PATCH_ERR_HIP; }
    if (st != PATCH_OK) {
        patch_free(P);
        return st;
    }
    *out = P;
    return PATCH_OK;
}

// Which kernel a pass of `rows` rows takes, and in how many K chunks.  Three kernels share up to 64 rows: the strip kernel
// (gemm_decode.hip: 16 features per workgroup), mid_kernel (64 features) and batch_kernel (128 features, and alone up to 128 rows).  A
// launch is bound by what one compute unit draws, so each is priced as
//     base + round (rounds - 1) + rounds x K-steps per workgroup x (step + per_row rows) x (1 + fill min(1, workgroups / compute units)) x (1 + sparse (f - 1/2)),
// rounds = ceil(workgroups / compute units), f = share of 2:4 tiles, and never less than its weights at 6.6 TB/s.  A split costs a second
// launch (2.2 us behind mid_kernel, 2.7 behind batch_kernel) and its partial sums twice through memory (5 TB/s).  Fitted to 24 weights from
// 128 x 4096 to 128256 x 1024 and 12 sets, both mask tiles, f = 0, 1/2 and 1, 22 row counts (860 - 4100 launches per line; rms error
// 4 - 7 %).  The row ranges are those of the kernels' row blocks: 17 - 32 rows of the strip kernel cost little more than 16 (4096 x 4096, f = 1/2,
// 16 / 17 / 24 / 32 rows 8.0 / 8.9 / 10.6 / 12.1 us, 33 rows 15.2; mid_kernel 13.5 / 14.4 / 15.6 / 16.8 and 19.9).  f tells the kernels apart: at 16 rows three
// 4096 x 4096 take mid_kernel 19.8 / 16.1 / 12.3 us at f = 0 / 1/2 / 1 and the strip kernel 22.9 / 19.4 / 17.5.
struct PassPrice { int rows; double base, step, per_row, fill, round, sparse; };
constexpr PassPrice kStripPrice[] = {{16, 2.5, 0.032, 0.0023, 0.24, 0.35, -0.23}, {32, 2.9, 0.045, 0.0026, 0.06, 0.4, -0.12}, {64, 3.5, 0.082, 0.0024, 0.07, 0.5, -0.03}};
constexpr PassPrice kMidPrice[] = {{16, 2.6, 0.120, 0.0017, 0.47, 1.5, -0.45}, {32, 3.2, 0.125, 0.0020, 0.40, 2.0, -0.40}, {64, 4.3, 0.143, 0.0024, 0.28, 3.3, -0.31}};
constexpr PassPrice kBatchPrice[] = {{16, 2.4, 0.257, 0.0005, 0.39, 0.0, -0.30}, {32, 2.7, 0.244, 0.0012, 0.40, 0.8, -0.29}, {64, 3.2, 0.237, 0.0017, 0.31, 3.2, -0.20},
                                     {80, 3.7, 0.392, 0.0005, 0.14, 4.0, 0.0},   {96, 4.1, 0.452, 0.0004, 0.10, 4.0, 0.03},  {128, 4.7, 0.570, 0.0004, 0.10, 4.0, 0.03}};

struct DecodePlan { int kernel, chunks; double us; int deal = 1; };   // kernel: 0 strip, 1 mid, 2 batch; rows dealt over up to `deal` workgroups (rows_each)
struct DecodeShape { int64_t N; int strips, groups64, groups128; size_t payload; int count; };   // of a weight or a whole set

static double pass_us(const PassPrice* p, const GemmArgs& a, const DecodeShape& d, int all_rows, int deal, int groups, int chunks, double second) {
    const int rows = rows_each(all_rows, deal);
    while (rows > p->rows) ++p;
    const int64_t wg = (int64_t)groups * chunks * rows_deals(all_rows, rows), rounds = (wg + a.n_cus - 1) / a.n_cus;
    const double fill = wg < a.n_cus ? (double)wg / a.n_cus : 1.0, weights = (double)d.payload / 6.6e6;
    const double t = (double)rounds * a.K / kStepCols / chunks * (p->step + p->per_row * rows) * (1.0 + p->fill * fill) * (1.0 + p->sparse * (0.01 * a.sparse_pct - 0.5));
    return p->base + p->round * (double)(rounds - 1) + (t > weights ? t : weights) + (chunks > 1 ? second + 2.0 * chunks * all_rows * (double)d.N * 4.0 / 5.0e6 : 0.0);
}

// The cheapest of the three; up to 7 rows (11 for a single weight) always the strip kernel, whose X is small then.  mid_kernel has to be 0.3 us ahead
// of it, batch_kernel 0.7 of both; of the strip kernel with its rows dealt (below) mid_kernel may be 0.15 behind.  only_wide: batch_kernel, in its best number of chunks.
// In a call of 17 .. 64 rows the strip kernel and mid_kernel may deal the blocks of 16 rows over 2 or 4 workgroups per feature group: a weight of few groups leaves compute units idle
// while each of its workgroups draws all of X.  The weights are read by every deal, from one L2 (deal_units).  The same prices hold: 5128 dealt calls over 48 weights and
// sets, both mask tiles, f = 0, 1/2 and 1, 17 - 64 rows, hot and cold weights, took 0.70 of the time of the best undealt choice, one of them 6 % more (8192 x 2048, f = 0,
// 44 rows with a workspace: 13.1 us, batch_kernel in 4 chunks 12.1).  f = 1/2, mask tile 128, 64 rows, undealt -> dealt: three 896 x 896 7.2 -> 4.8, 896 x 4864
// 21.3 -> 8.6, 4096 x 4096 20.1 -> 13.1, 4864 x 13824 at 40 rows 59.6 -> 39.9 us.  (A call of more rows is passes of 64 and the rest, and takes the prefill path
// where that is cheaper; dealing its passes was not measured.)
static DecodePlan decode_plan(const GemmArgs& a, const DecodeShape& d, int rows, bool only_wide = false) {
    DecodePlan best = {0, 1, 0.0};
    if (!only_wide) {
        best.us = pass_us(kStripPrice, a, d, rows, 1, d.strips, 1, 0.0);
        if (rows < (d.count > 1 ? 8 : 12)) return best;
        for (int deal = 1, last = 0; deal <= 4; deal *= 2) {
            const int each = rows_each(rows, deal);
            if (deal > 1 && (rows <= 16 || a.M > kDecodeRows || each == last)) break;
            last = each;
            const auto take = [&](int kernel, int chunks, double us, double ahead) {
                if (us + ahead < best.us) { best = DecodePlan{kernel, chunks, us}; best.deal = deal; }
            };
            if (deal > 1) take(0, 1, pass_us(kStripPrice, a, d, rows, deal, d.strips, 1, 0.0), 0.0);
            const auto ahead = [&]() { return best.kernel != 0 ? 0.0 : best.deal == 1 ? 0.3 : -0.15; };
            take(1, 1, pass_us(kMidPrice, a, d, rows, deal, d.groups64, 1, 2.2), ahead());
            if (const int c = d.count == 1 && rows > 16 ? mid_split(a, rows, 0, (int)rows_deals(rows, each)) : 1; c > 1)
                take(1, c, pass_us(kMidPrice, a, d, rows, deal, d.groups64, c, 2.2), ahead());
        }
    }
    // (at most 8 chunks of at least four units of 128 columns; beyond one workgroup per compute unit a split only adds partial sums)
    const size_t per_chunk = (size_t)rows * (size_t)d.N * sizeof(float);
    const int fit = a.ws ? (int)(a.ws_bytes / per_chunk < 8 ? a.ws_bytes / per_chunk : 8) : 1;
    DecodePlan wide = {2, 1, pass_us(kBatchPrice, a, d, rows, 1, d.groups128, 1, 0.0)};
    for (int c = 2; c <= fit && d.groups128 * c <= a.n_cus && c * 512 <= a.K; ++c) {
        const double t = pass_us(kBatchPrice, a, d, rows, 1, d.groups128, c, 2.7);
        if (t < wide.us) wide = DecodePlan{2, c, t};
    }
    return only_wide || wide.us + 0.7 < best.us ? wide : best;
}

// batch_kernel on request (variant 7): `requested` K chunks as far as they exist and the workspace holds them, 0 = the plan's
static DecodePlan batch_plan(const GemmArgs& a, const DecodeShape& d, int rows, int requested) {
    if (requested == 0) return decode_plan(a, d, rows, true);
    const size_t per_chunk = (size_t)rows * (size_t)d.N * sizeof(float);
    int c = requested;
    if (c > (a.K + 127) / 128) c = (int)((a.K + 127) / 128);
    const size_t fit = a.ws ? a.ws_bytes / per_chunk : 1;
    if ((size_t)c > fit) c = (int)fit;
    return DecodePlan{2, c < 1 ? 1 : c, 0.0};
}

static DecodeShape decode_shape(const patch_packed* P) {
    return DecodeShape{P->N, (int)(P->N / 16), (int)(P->N / 64), (int)((P->N + 127) / 128), P->payload_bytes, 1};
}

// us a prefill launch over all weights of a set is estimated to take (a.N: the first weight's)
static double set_prefill_us(const GemmArgs& a, const DecodeShape& d, const int64_t* N) {
    if (d.count == 1) return prefill_estimate(a);
    if (prefill_wreg_supports(a)) return prefill_set_estimate(a, N, d.count);
    // (beyond the limits of the set launch the weights go one by one: priced as one launch after the other)
    double us = 0.0;
    for (int i = 0; i < d.count; ++i) {
        GemmArgs one = a;
        one.N = N[i];
        us += prefill_estimate(one);
    }
    return us;
}

// What AUTO stands for: passes, each streaming the whole weight, or one prefill launch, by the estimate of both (prefill_estimate,
// decode_plan).  d: the weight or the whole set; N[i]: features of weight i; nothing_asked: neither variant nor split_k, so that 65 .. 128
// rows may go in one pass of batch_kernel.
//   up to 32 rows, sets up to 64: a pass
//   a single weight of 33 .. 64 rows: a pass, or the prefill launch where the weight is wider than the chip (f = 1/2, 64 rows: 128256 x 1024
//     51 us in a pass, 39 on the prefill kernel; 32896 x 4096 59 and 52; 20480 x 4096 31 and 50, split over a workspace 30)
//   65 .. 128 rows: one pass where it is estimated 2 % ahead of the prefill launch - whose K split writes and reads its partial products more
//     often, or which leaves compute units idle - and, without a workspace, of two passes.  f = 1/2, 80 / 128 rows, prefill -> pass: three
//     4096 x 4096 32.7 / 34.7 -> 26.0 / 34.8 us, gate and up of 5120 / 13824 59.6 / 64.0 -> 46.6 / 61.6; at f = 1 the prefill launch gains
//     more from its 2:4 steps (two 28672 x 4096, 80 rows 64 us against 73)
//   beyond, with a workspace for two slices: prefill, whose K split fills the chip at any number of rows; without, the cheaper side
struct AutoChoice { int path; bool one_pass; DecodePlan pass; };
static AutoChoice auto_choice(const GemmArgs& a, const DecodeShape& d, const int64_t* N, bool nothing_asked) {
    const int64_t M = a.M;
    const bool ws = a.ws && a.ws_bytes >= 2 * (size_t)M * (size_t)N[0] * sizeof(float);
    AutoChoice c = {PATCH_PATH_DECODE, false, {2, 1, 0.0}};
    if (M <= (d.count > 1 ? kDecodeRows : 32)) return c;
    const bool one_pass = nothing_asked && M > kDecodeRows && M <= kBatchRows;
    if (ws && M > kDecodeRows && !one_pass) { c.path = PATCH_PATH_PREFILL; return c; }
    const double prefill_us = set_prefill_us(a, d, N);
    double passes_us = 0.0;
    if (!ws || M <= kDecodeRows) {
        const int64_t full = M / kDecodeRows, rest = M % kDecodeRows;
        passes_us = (full ? (double)full * decode_plan(a, d, kDecodeRows).us : 0.0) + (rest ? decode_plan(a, d, (int)rest).us : 0.0);
    }
    if (one_pass) {
        c.pass = decode_plan(a, d, (int)M, true);
        c.one_pass = 1.02 * c.pass.us < (ws ? prefill_us : std::min(prefill_us, passes_us));
    }
    if (!c.one_pass && (passes_us == 0.0 || prefill_us <= passes_us)) c.path = PATCH_PATH_PREFILL;
    return c;
}

// Test hooks (kernels.h)
int patch_test_schedule(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes, int* kernel, int* chunks) {
    int deals[8];
    return patch_test_schedule_deals(M, count, N, K, tile, sparse_pct, ws_bytes, kernel, chunks, deals);
}

int patch_test_schedule_deals(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes, int* kernel, int* chunks, int* deals) {
    if (!N || !kernel || !chunks || !deals || M < 1 || count < 1 || count > kMaxMany || sparse_pct < 0 || sparse_pct > 100) return -1;
    GemmArgs a = {};
    a.M = M; a.N = N[0]; a.K = K;
    a.tile = tile; a.Tk = (int)(K / tile);
    a.n_cus = 256;
    a.sparse_pct = sparse_pct;
    if (ws_bytes) { a.ws = reinterpret_cast<float*>(16); a.ws_bytes = ws_bytes; }
    DecodeShape d = {0, 0, 0, 0, 0, count};
    for (int i = 0; i < count; ++i) {
        if (check_shape(N[i], K, tile) != PATCH_OK) return -1;
        const DecodeShape w = {N[i], (int)(N[i] / 16), (int)(N[i] / 64), (int)((N[i] + 127) / 128), (size_t)(2.0 * (double)N[i] * (double)K * (1.0 - 0.07 / 16.0 * sparse_pct)), 1};
        d.N += w.N; d.strips += w.strips; d.groups64 += w.groups64; d.groups128 += w.groups128; d.payload += w.payload;
    }
    const AutoChoice c = auto_choice(a, d, N, true);
    if (c.one_pass || c.path == PATCH_PATH_PREFILL) {
        kernel[0] = c.one_pass ? c.pass.kernel : 3;
        chunks[0] = c.one_pass ? c.pass.chunks : 1;
        deals[0] = 1;
        if (int split = 1; kernel[0] == 3 && count == 1 && prefill_prefers_128_rows(a, &split)) {
            kernel[0] = 4;
            chunks[0] = split;
        }
        return 1;
    }
    if (M > 8 * kDecodeRows) return -1;
    int n = 0;
    for (int64_t m0 = 0; m0 < M; m0 += kDecodeRows, ++n) {
        const int rows = (int)(M - m0 < kDecodeRows ? M - m0 : kDecodeRows);
        const DecodePlan plan = decode_plan(a, d, rows);
        kernel[n] = plan.kernel;
        chunks[n] = plan.chunks;
        deals[n] = (int)rows_deals(rows, rows_each(rows, plan.deal));
    }
    return n;
}

// a prefill-path launch as patch_test_schedule describes it; false = bad arguments
static bool test_prefill_args(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes, GemmArgs* a) {
    if (!N || M < 1 || count < 1 || count > kMaxMany || sparse_pct < 0 || sparse_pct > 100) return false;
    for (int i = 0; i < count; ++i)
        if (check_shape(N[i], K, tile) != PATCH_OK) return false;
    *a = {};
    a->M = M; a->N = N[0]; a->K = K;
    a->tile = tile; a->Tk = (int)(K / tile);
    a->n_cus = 256;
    a->sparse_pct = sparse_pct;
    if (ws_bytes) { a->ws = reinterpret_cast<float*>(16); a->ws_bytes = ws_bytes; }
    return true;
}

int patch_test_prefill128_split(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes) {
    GemmArgs a;
    return test_prefill_args(M, count, N, K, tile, sparse_pct, ws_bytes, &a) ? prefill_r128_split(a, N, count) : -1;
}

int patch_test_last_round(int64_t M, int count, const int64_t* N, int64_t K, int tile, int sparse_pct, size_t ws_bytes, int* slices, int* halves) {
    GemmArgs a;
    if (!slices || !halves || !test_prefill_args(M, count, N, K, tile, sparse_pct, ws_bytes, &a) || !prefill_wreg_supports(a)) return -1;
    int64_t tiles = 0;
    for (int i = 0; i < count; ++i) tiles += (N[i] + 255) / 256 * ((M + 255) / 256);
    const LastRound r = prefill_wreg_last_round((int)tiles, a);
    *slices = r.slices;
    *halves = r.halves;
    return r.tail;
}

// the set of a test hook's weights, by blocks of 256 features; false = bad arguments
static bool test_prefill_set(const void* X, int64_t M, const patch_packed* const* P, void* const* Y, int count, int y_bf16, void* workspace,
                             size_t workspace_bytes, GemmArgs* a, WeightSet* set) {
    if (!X || !P || !Y || M < 1 || count < 1 || count > kMaxMany) return false;
    *a = {};
    *set = {};
    a->X = static_cast<const uint16_t*>(X);
    a->M = M; a->K = P[0]->K; a->tile = P[0]->tile; a->Tk = P[0]->Tk; a->n_cus = P[0]->n_cus;
    a->ybf16 = y_bf16 ? 1 : 0;
    a->ws = static_cast<float*>(workspace);
    a->ws_bytes = workspace_bytes;
    for (int i = 0; i < count; ++i) {
        if (!P[i] || !Y[i] || P[i]->K != a->K || P[i]->tile != a->tile) return false;
        set->payload[i] = P[i]->d_payload; set->table[i] = P[i]->d_table; set->Y[i] = static_cast<float*>(Y[i]); set->N[i] = P[i]->N;
        set->first[i] = set->units;
        set->units += (int)((P[i]->N + 255) / 256);
        a->N += P[i]->N;
    }
    set->count = count;
    return true;
}

int patch_test_prefill128(const void* X, int64_t M, const patch_packed* const* P, void* const* Y, int count, int split, int y_bf16, void* workspace,
                          size_t workspace_bytes, void* stream) {
    GemmArgs a;
    WeightSet set;
    if (!test_prefill_set(X, M, P, Y, count, y_bf16, workspace, workspace_bytes, &a, &set) || split < 1 || split > 16 || split > a.Tk) return -1;
    if (split > 1 && (!workspace || workspace_bytes / sizeof(float) / (size_t)split < (size_t)M * (size_t)a.N)) return -1;
    launch_prefill_r128(a, set, split, static_cast<hipStream_t>(stream));
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int patch_test_prefill_last_round(const void* X, int64_t M, const patch_packed* const* P, void* const* Y, int count, int halves, int slices, int y_bf16,
                                  void* workspace, size_t workspace_bytes, void* stream) {
    GemmArgs a;
    WeightSet set;
    if (!test_prefill_set(X, M, P, Y, count, y_bf16, workspace, workspace_bytes, &a, &set) || !prefill_wreg_supports(a)) return -1;
    const int tiles_m = (int)((M + 255) / 256), tail = set.units * tiles_m % a.n_cus;
    if (halves >= 0 && (slices < 1 || slices > 8 || slices > a.Tk || (halves == 0 && slices == 1) || tail == 0 || set.units * tiles_m < a.n_cus)) return -1;
    if (halves >= 0 && slices > 1 && (!workspace || workspace_bytes < (size_t)tail * slices * 256 * 256 * sizeof(float))) return -1;
    launch_prefill_wreg_rounds(a, set, tiles_m, halves < 0 ? LastRound{0, 1, false} : LastRound{tail, slices, halves != 0}, static_cast<hipStream_t>(stream));
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int64_t patch_test_map_args(const uint8_t* map, int n, uint32_t before, uint32_t* out) {
    if (!map || !out || n < 1 || n > kMapTiles) return -1;
    TileMapArgs a;
    before = fill_map_args(&a, map, n, before);
    memcpy(out, a.g, (size_t)(n + 63) / 64 * sizeof a.g[0]);
    return before;
}

int patch_test_deal_units(int units, int deals, int n_cus) { return units < 1 || deals < 1 || n_cus < 8 ? -1 : (int)deal_units(units, (unsigned)deals, n_cus); }

patch_status patch_gemm_ex(const void* X, int64_t M, const patch_packed* P, void* Y, void* stream, const patch_gemm_opts* opts) {
    if (!X || !P || !Y || M < 0) return PATCH_ERR_ARG;
    if (!aligned16(X) || !aligned16(Y)) return PATCH_ERR_ARG;
    int path = PATCH_PATH_AUTO, split_k = 0, variant = 0;
    if (opts) { path = opts->path; split_k = opts->split_k; variant = opts->variant; }
    if (path < PATCH_PATH_AUTO || path > PATCH_PATH_PREFILL || split_k < 0 || split_k > 16 || variant < 0) return PATCH_ERR_ARG;
    if (opts && opts->workspace && !aligned16(opts->workspace)) return PATCH_ERR_ARG;
    if (M == 0) return PATCH_OK;  // an empty batch: nothing to launch, Y has no rows
    hipStream_t s = static_cast<hipStream_t>(stream);
    GemmArgs a;
    a.X = static_cast<const uint16_t*>(X);
    a.M = M; a.N = P->N; a.K = P->K;
    a.tile = P->tile; a.Tn = P->Tn; a.Tk = P->Tk;
    a.payload = P->d_payload; a.table = P->d_table;
    a.Y = static_cast<float*>(Y);
    a.n_cus = P->n_cus;
    a.sparse_pct = (int)(100 * P->n_sparse / ((int64_t)P->Tn * P->Tk));
    if (opts && opts->workspace) { a.ws = static_cast<float*>(opts->workspace); a.ws_bytes = opts->workspace_bytes; }
    a.ybf16 = (opts && opts->y_bf16) ? 1 : 0;
    WeightSet one = {};
    one.payload[0] = a.payload; one.table[0] = a.table; one.Y[0] = a.Y; one.N[0] = a.N;
    one.count = 1;
    const DecodeShape d = decode_shape(P);
    if (path == PATCH_PATH_AUTO) {
        const AutoChoice c = auto_choice(a, d, &P->N, variant == 0 && split_k == 0);
        path = c.path;
        if (c.one_pass) {
            one.units = d.groups128;
            launch_batch_set(a, one, 0, (int)M, c.pass.chunks, s);
            HIP_TRY(hipGetLastError());
            return PATCH_OK;
        }
    }
    if (path == PATCH_PATH_DECODE) {
        for (int64_t m0 = 0; m0 < M; m0 += (variant == 7 ? kBatchRows : kDecodeRows)) {
            const int rows = (int)((M - m0 < (variant == 7 ? kBatchRows : kDecodeRows)) ? M - m0 : (variant == 7 ? kBatchRows : kDecodeRows));
            DecodePlan plan = {0, 1, 0.0};
            if (variant == 4) plan = DecodePlan{1, mid_split(a, rows, split_k), 0.0};
            else if (variant == 7) plan = batch_plan(a, d, rows, split_k);
            else if (variant == 0 && split_k == 0) plan = decode_plan(a, d, rows);
            one.units = plan.kernel == 2 ? d.groups128 : d.groups64;
            if (plan.kernel == 2) launch_batch_set(a, one, m0, rows, plan.chunks, s);
            else if (plan.kernel == 1) launch_mid_set(a, one, m0, rows, plan.chunks, s, plan.deal);
            else launch_decode(a, m0, rows, split_k, variant, s, plan.deal);
        }
    } else {
        launch_prefill(a, variant, split_k, s);
    }
    HIP_TRY(hipGetLastError());
    return PATCH_OK;
}

patch_status patch_tune_all(const void* X, int64_t M, const patch_packed* P, void* Y, void* workspace, size_t workspace_bytes,
                            void* stream, int reps, patch_tune_result* results, size_t cap, size_t* count) {
    if (!X || !P || !Y || !results || !count || M <= 0 || reps < 1) return PATCH_ERR_ARG;
    if (!aligned16(X) || !aligned16(Y) || (workspace && !aligned16(workspace))) return PATCH_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    std::vector<patch_gemm_opts> cand;
    auto add = [&](int path, int split_k, int variant, bool ws) {
        cand.push_back(patch_gemm_opts{path, split_k, variant, ws ? workspace : nullptr, ws ? workspace_bytes : 0, 0});
    };
    const int steps = P->Tk * (P->tile / kStepCols);
    if (M <= 256) {  // every pass of 64 rows streams the whole weight again: no contender beyond that
        add(PATCH_PATH_DECODE, 0, 0, false);
        add(PATCH_PATH_DECODE, 0, 2, false);   // 8 K-steps per wavefront
        add(PATCH_PATH_DECODE, 0, 3, false);   // 4 K-steps per wavefront
        if (M <= 8) {                          // X loads: two per step / one for several steps
            add(PATCH_PATH_DECODE, 0, 5, false);
            add(PATCH_PATH_DECODE, 0, 6, false);
        }
        for (int kw : {2, 4, 8, 16})           // wavefronts per workgroup
            for (int v : {2, 3})
                if (kw * (v == 2 ? 8 : 4) <= 2 * steps && (kw <= 8 || v == 3)) add(PATCH_PATH_DECODE, kw, v, false);
        if (M >= 12 && workspace) add(PATCH_PATH_DECODE, 0, 0, true);   // what AUTO takes of the decode path: K chunks and dealt rows together are no other candidate's
        if (M >= 12) {  // the 64-features-per-wavefront kernel, unsplit and with K-chunks over the workspace
            add(PATCH_PATH_DECODE, 0, 4, false);
            const size_t per_slice = (size_t)(M < kDecodeRows ? M : kDecodeRows) * (size_t)P->N * sizeof(float);
            if (workspace)
                for (int sk : {2, 3, 4, 6, 8})
                    if ((size_t)sk * per_slice <= workspace_bytes && sk <= P->Tk) add(PATCH_PATH_DECODE, sk, 4, true);
            add(PATCH_PATH_DECODE, 1, 7, false);   // 128 features per workgroup, unsplit and in the planned number of chunks
            if (workspace) add(PATCH_PATH_DECODE, 0, 7, true);
        }
    }
    const size_t per_slice = (size_t)M * (size_t)P->N * sizeof(float);
    const int tiles_per_slice = 512 / P->tile;   // K slices of at least 512 columns
    if (P->tile == 128) {
        add(PATCH_PATH_PREFILL, 1, 0, false);   // 256 x 256, one wavefront per SIMD
        add(PATCH_PATH_PREFILL, 1, 2, false);   // 256 x 256, two wavefronts per SIMD
        add(PATCH_PATH_PREFILL, 1, 1, false);   // 128 x 128: the small execution tile
        if (workspace) add(PATCH_PATH_PREFILL, 0, 0, true);   // automatic: may split a part-filled last round only
        if (workspace)
            for (int sk : {2, 3, 4, 6, 8, 12, 16})
                if ((size_t)sk * per_slice <= workspace_bytes && sk * 2 <= P->Tk) add(PATCH_PATH_PREFILL, sk, 0, true);
    } else {
        add(PATCH_PATH_PREFILL, 1, 0, false);   // 256 x 256 with the weights in registers (the tile-64 default)
        add(PATCH_PATH_PREFILL, 1, 2, false);   // 256 x 256 LDS-staged
        add(PATCH_PATH_PREFILL, 1, 1, false);   // 128 x 128: the small execution tile
        if (workspace) add(PATCH_PATH_PREFILL, 0, 0, true);   // automatic
        if (workspace)
            for (int sk : {2, 3, 4, 6, 8})
                if ((size_t)sk * per_slice <= workspace_bytes && sk * 4 <= P->Tk) add(PATCH_PATH_PREFILL, sk, 0, true);
    }
    if (M <= 4096) {   // 256 features x 128 rows per workgroup: beyond a few thousand rows never ahead
        for (int v : {4, 5}) {   // LDS-staged; weights in registers
            add(PATCH_PATH_PREFILL, 1, v, false);
            if (workspace)
                for (int sk : {2, 3, 4, 6, 8})
                    if ((size_t)sk * per_slice <= workspace_bytes && sk * tiles_per_slice <= P->Tk) add(PATCH_PATH_PREFILL, sk, v, true);
        }
    }
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    if (hipError_t e = hipEventCreate(&e1); e != hipSuccess) { (void)hipEventDestroy(e0); g_last_hip_error = (int)e; return PATCH_ERR_HIP; }
    patch_status st = PATCH_OK;
    for (size_t i = 0; i < cand.size() && st == PATCH_OK; ++i) {
        for (int r = 0; r < 2 && st == PATCH_OK; ++r) st = patch_gemm_ex(X, M, P, Y, stream, &cand[i]);
        if (st != PATCH_OK) break;
        hipError_t e = hipEventRecord(e0, s);
        for (int r = 0; r < reps && st == PATCH_OK; ++r) st = patch_gemm_ex(X, M, P, Y, stream, &cand[i]);
        if (e == hipSuccess) e = hipEventRecord(e1, s);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        if (e != hipSuccess) { g_last_hip_error = (int)e; st = PATCH_ERR_HIP; break; }
        if (i < cap) results[i] = patch_tune_result{cand[i], ms * 1000.f / (float)reps};
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != PATCH_OK) return st;
    *count = cand.size();
    return PATCH_OK;
}

patch_status patch_tune(const void* X, int64_t M, const patch_packed* P, void* Y, void* workspace, size_t workspace_bytes,
                        void* stream, int reps, patch_gemm_opts* best, float* best_us) {
    if (!best) return PATCH_ERR_ARG;
    constexpr size_t kCap = 64;
    patch_tune_result res[kCap];
    size_t n = 0;
    const patch_status st = patch_tune_all(X, M, P, Y, workspace, workspace_bytes, stream, reps, res, kCap, &n);
    if (st != PATCH_OK) return st;
    if (n > kCap) n = kCap;
    size_t bi = 0;
    for (size_t i = 1; i < n; ++i)
        if (res[i].us < res[bi].us) bi = i;
    *best = res[bi].opts;
    if (best_us) *best_us = res[bi].us;
    // leave the product of the chosen schedule in Y
    return patch_gemm_ex(X, M, P, Y, stream, best);
}

// ---- table of tuned schedules
struct TuneKey {
    int64_t bucket, N, K, n_sparse;
    int tile;
    bool operator<(const TuneKey& o) const {
        return std::tie(bucket, N, K, n_sparse, tile) < std::tie(o.bucket, o.N, o.K, o.n_sparse, o.tile);
    }
};
struct TuneEntry { int path, split_k, variant, y_bf16; bool uses_ws; };
struct patch_tune_table {
    mutable std::mutex mu;
    std::map<TuneKey, TuneEntry> entries;
};

int64_t patch_tune_bucket(int64_t M) {
    if (M <= 1) return 1;
    int64_t b = 1;
    while (b < M && b < ((int64_t)1 << 62)) b <<= 1;
    return b;
}

patch_status patch_tune_table_create(patch_tune_table** out) {
    if (!out) return PATCH_ERR_ARG;
    patch_tune_table* t = new (std::nothrow) patch_tune_table();
    if (!t) return PATCH_ERR_ALLOC;
    *out = t;
    return PATCH_OK;
}

void patch_tune_table_destroy(patch_tune_table* t) { delete t; }

size_t patch_tune_table_size(const patch_tune_table* t) {
    if (!t) return 0;
    std::lock_guard<std::mutex> lock(t->mu);
    return t->entries.size();
}

static bool tune_key_ok(int64_t M, int64_t N, int64_t K, int tile, int64_t ns) {
    return M >= 1 && ns >= 0 && check_shape(N, K, tile) == PATCH_OK && ns <= (N / tile) * (K / tile);
}

patch_status patch_tune_table_put(patch_tune_table* t, int64_t M, int64_t N, int64_t K, int tile, int64_t n_sparse_tiles,
                                  const patch_gemm_opts* opts) {
    if (!t || !opts || !tune_key_ok(M, N, K, tile, n_sparse_tiles)) return PATCH_ERR_ARG;
    if (opts->path < PATCH_PATH_AUTO || opts->path > PATCH_PATH_PREFILL || opts->split_k < 0 || opts->split_k > 16 || opts->variant < 0)
        return PATCH_ERR_ARG;
    const TuneKey k{patch_tune_bucket(M), N, K, n_sparse_tiles, tile};
    const TuneEntry e{opts->path, opts->split_k, opts->variant, opts->y_bf16 ? 1 : 0, opts->workspace != nullptr};
    std::lock_guard<std::mutex> lock(t->mu);
    try { t->entries[k] = e; } catch (...) { return PATCH_ERR_ALLOC; }
    return PATCH_OK;
}

patch_status patch_tune_table_get(const patch_tune_table* t, int64_t M, int64_t N, int64_t K, int tile, int64_t n_sparse_tiles,
                                  void* workspace, size_t workspace_bytes, patch_gemm_opts* out) {
    if (!t || !out || !tune_key_ok(M, N, K, tile, n_sparse_tiles)) return PATCH_ERR_ARG;
    const TuneKey k{patch_tune_bucket(M), N, K, n_sparse_tiles, tile};
    std::lock_guard<std::mutex> lock(t->mu);
    const auto it = t->entries.find(k);
    if (it == t->entries.end()) return PATCH_ERR_NOT_FOUND;
    const TuneEntry& e = it->second;
    if (e.uses_ws && !workspace) return PATCH_ERR_NOT_FOUND;
    *out = patch_gemm_opts{e.path, e.split_k, e.variant, e.uses_ws ? workspace : nullptr, e.uses_ws ? workspace_bytes : 0, e.y_bf16};
    return PATCH_OK;
}

patch_status patch_tune_table_export(const patch_tune_table* t, patch_tune_entry* entries, size_t cap, size_t* count) {
    if (!t || !count || (!entries && cap)) return PATCH_ERR_ARG;
    std::lock_guard<std::mutex> lock(t->mu);
    *count = t->entries.size();
    if (!entries) return PATCH_OK;          // a size query
    if (cap < t->entries.size()) return PATCH_ERR_SIZE;
    size_t i = 0;
    for (const auto& kv : t->entries) {
        const TuneKey& k = kv.first;
        const TuneEntry& e = kv.second;
        entries[i++] = patch_tune_entry{k.bucket, k.N, k.K, k.n_sparse, k.tile, e.path, e.split_k, e.variant, e.y_bf16, e.uses_ws ? 1 : 0};
    }
    return PATCH_OK;
}

patch_status patch_tune_table_import(patch_tune_table* t, const patch_tune_entry* entries, size_t count) {
    if (!t || (!entries && count)) return PATCH_ERR_ARG;
    // all or nothing: every entry is checked before the first is stored
    for (size_t i = 0; i < count; ++i) {
        const patch_tune_entry& e = entries[i];
        if (!tune_key_ok(e.m_bucket, e.N, e.K, e.tile, e.n_sparse_tiles) || patch_tune_bucket(e.m_bucket) != e.m_bucket) return PATCH_ERR_ARG;
        if (e.path < PATCH_PATH_AUTO || e.path > PATCH_PATH_PREFILL || e.split_k < 0 || e.split_k > 16 || e.variant < 0) return PATCH_ERR_ARG;
    }
    std::lock_guard<std::mutex> lock(t->mu);
    try {
        for (size_t i = 0; i < count; ++i) {
            const patch_tune_entry& e = entries[i];
            t->entries[TuneKey{e.m_bucket, e.N, e.K, e.n_sparse_tiles, e.tile}] =
                TuneEntry{e.path, e.split_k, e.variant, e.y_bf16 ? 1 : 0, e.uses_workspace != 0};
        }
    } catch (...) { return PATCH_ERR_ALLOC; }
    return PATCH_OK;
}

patch_status patch_tune_layer(patch_tune_table* t, const void* X_decode, int64_t M_decode, const void* X_prefill, int64_t M_prefill,
                              const patch_packed* P, void* Y, void* workspace, size_t workspace_bytes, void* stream, int reps) {
    if (!t || !P || !X_decode || !X_prefill || M_decode < 1 || M_prefill < 1) return PATCH_ERR_ARG;
    // the decode input first, then the prefill input, both from the one packed weight
    const void* xs[2] = {X_decode, X_prefill};
    const int64_t ms[2] = {M_decode, M_prefill};
    for (int i = 0; i < 2; ++i) {
        patch_gemm_opts best;
        patch_status st = patch_tune(xs[i], ms[i], P, Y, workspace, workspace_bytes, stream, reps, &best, nullptr);
        if (st != PATCH_OK) return st;
        st = patch_tune_table_put(t, ms[i], P->N, P->K, P->tile, P->n_sparse, &best);
        if (st != PATCH_OK) return st;
    }
    return PATCH_OK;
}

// Bytes of workspace that let a product run as if given any amount; no less than the kernels in 256-row tiles would use in place of
// prefill_kernel_r128.  slices_only: what patch_gemm_static accepts and refuses by, whatever it launches: the slices of 256-row tiles - mask tile 128: of
// the whole product or of the last round (prefill_wreg_tail_bytes); mask tile 64: of the whole product, as prefill_kernel_areg would make them.
static size_t workspace_need(int64_t M, const patch_packed* P, const patch_gemm_opts* opts, bool slices_only) {
    if (!P || M <= 0) return 0;
    int path = PATCH_PATH_AUTO, split_k = 0, variant = 0;
    if (opts) { path = opts->path; split_k = opts->split_k; variant = opts->variant; }
    GemmArgs a = {};
    a.M = M; a.N = P->N; a.K = P->K;
    a.tile = P->tile; a.Tn = P->Tn; a.Tk = P->Tk;
    a.n_cus = P->n_cus;
    a.sparse_pct = (int)(100 * P->n_sparse / ((int64_t)P->Tn * P->Tk));
    a.ws = reinterpret_cast<float*>(16);  // "enough": ask for the unconstrained choice
    a.ws_bytes = ~(size_t)0;
    // 65 .. 128 rows: what one pass would use, and no less than the prefill launch it stands in for (below)
    size_t least = 0;
    if (path == PATCH_PATH_AUTO) {
        const DecodeShape d = decode_shape(P);
        const AutoChoice c = auto_choice(a, d, &P->N, variant == 0 && split_k == 0);
        path = c.path;
        if (c.one_pass) {
            path = PATCH_PATH_PREFILL;
            if (c.pass.chunks > 1) least = (size_t)c.pass.chunks * (size_t)M * (size_t)P->N * sizeof(float);
        }
    }
    if (path == PATCH_PATH_DECODE) {
        // a pass may cut K into chunks over the workspace; the full passes and the last one each have a number of their own
        const int64_t pass = variant == 7 ? kBatchRows : kDecodeRows;
        size_t most = 0;
        for (const int64_t r : {M < pass ? M : pass, M % pass}) {
            const int rows = (int)r;
            if (rows == 0) continue;
            int chunks = 1;
            if (variant == 4) chunks = mid_split(a, rows, split_k);
            else if (variant == 7) chunks = batch_plan(a, decode_shape(P), rows, split_k).chunks;
            else if (variant == 0 && split_k == 0) {
                // (from 17 rows at least what mid_kernel would take, whichever kernel the plan prefers: a caller that asked before
                // and one that asks now get no smaller a buffer)
                chunks = decode_plan(a, decode_shape(P), rows).chunks;
                if (rows > 16) chunks = std::max(chunks, mid_split(a, rows, 0));
            }
            if (chunks > 1) most = std::max(most, (size_t)chunks * (size_t)rows * (size_t)P->N * sizeof(float));
        }
        return most;
    }
    if (variant == 1) return 0;
    if (variant == 0 && split_k == 0 && !slices_only) {
        const int split = prefill_r128_split(a, &P->N, 1);   // (and no less than the launch would take without that kernel)
        if (split > 1) least = std::max(least, (size_t)split * (size_t)M * (size_t)P->N * sizeof(float));
    }
    if (variant == 0 && split_k == 0) {
        int split128 = 1;
        if (prefill_prefers_128_rows(a, &split128, slices_only)) return std::max(least, split128 > 1 ? (size_t)split128 * (size_t)M * (size_t)P->N * sizeof(float) : (size_t)0);
    }
    if (variant == 2 || variant == 4 || variant == 5 || (a.tile == 64 && (variant == 6 || slices_only)) || !prefill_wreg_supports(a)) {   // whole-launch K split only
        const int sl = prefill_lds_split(a, split_k, variant == 4 || variant == 5 ? 128 : 256);
        return std::max(least, sl > 1 ? (size_t)sl * (size_t)M * (size_t)P->N * sizeof(float) : (size_t)0);
    }
    const int s = prefill_wreg_split(a, split_k);
    if (s > 1) return std::max(least, (size_t)s * (size_t)M * (size_t)P->N * sizeof(float));
    if (split_k != 0) return 0;
    least = std::max(least, prefill_wreg_tail_bytes(a));   // K slices for the part-filled last round only
    if (slices_only) return least;
    const LastRound last = prefill_wreg_tail(a);
    return std::max(least, last.slices > 1 ? (size_t)last.slices * (size_t)last.tail * 256 * 256 * sizeof(float) : (size_t)0);
}

size_t patch_gemm_workspace_bytes(int64_t M, const patch_packed* P, const patch_gemm_opts* opts) { return workspace_need(M, P, opts, false); }

patch_status patch_gemm_many(const void* X, int64_t M, const patch_packed* const* P, void* const* Y, int count, void* stream,
                             const patch_gemm_opts* opts) {
    if (!X || !P || !Y || M < 0 || count < 1 || count > PATCH_MAX_MANY) return PATCH_ERR_ARG;
    static_assert(PATCH_MAX_MANY == kMaxMany, "header and kernels disagree");
    if (!aligned16(X)) return PATCH_ERR_ARG;
    for (int i = 0; i < count; ++i) {
        if (!P[i] || !Y[i] || !aligned16(Y[i])) return PATCH_ERR_ARG;
        if (P[i]->K != P[0]->K || P[i]->tile != P[0]->tile) return PATCH_ERR_SHAPE;
    }
    int path = PATCH_PATH_AUTO, split_k = 0, variant = 0;
    if (opts) { path = opts->path; split_k = opts->split_k; variant = opts->variant; }
    if (path < PATCH_PATH_AUTO || path > PATCH_PATH_PREFILL || split_k < 0 || split_k > 16 || variant < 0) return PATCH_ERR_ARG;
    if (M == 0) return PATCH_OK;
    if (count == 1) return patch_gemm_ex(X, M, P[0], Y[0], stream, opts);
    hipStream_t s = static_cast<hipStream_t>(stream);
    GemmArgs a = {};
    a.X = static_cast<const uint16_t*>(X);
    a.M = M; a.K = P[0]->K; a.N = P[0]->N;
    a.tile = P[0]->tile; a.Tk = P[0]->Tk;
    a.n_cus = P[0]->n_cus;
    {
        int64_t sparse = 0, tiles = 0;
        for (int i = 0; i < count; ++i) {
            if (!P[i]) return PATCH_ERR_ARG;
            sparse += P[i]->n_sparse;
            tiles += (int64_t)P[i]->Tn * P[i]->Tk;
        }
        a.sparse_pct = (int)(100 * sparse / tiles);
    }
    a.ybf16 = (opts && opts->y_bf16) ? 1 : 0;
    if (opts && opts->workspace && !aligned16(opts->workspace)) return PATCH_ERR_ARG;
    if (opts && opts->workspace) { a.ws = static_cast<float*>(opts->workspace); a.ws_bytes = opts->workspace_bytes; }
    DecodeSet set = {};
    int strips = 0;
    for (int i = 0; i < count; ++i) {
        set.payload[i] = P[i]->d_payload;
        set.table[i] = P[i]->d_table;
        set.Y[i] = static_cast<float*>(Y[i]);
        set.N[i] = P[i]->N;
        set.first[i] = strips;
        strips += (int)(P[i]->N / 16);
    }
    set.count = count;
    set.units = strips;
    // the same set in groups of 64 and of 128 features
    WeightSet wide64 = set, wide128 = set;
    DecodeShape d = {0, strips, 0, 0, 0, count};
    for (int i = 0; i < count; ++i) {
        const DecodeShape w = decode_shape(P[i]);
        wide64.first[i] = d.groups64;
        wide128.first[i] = d.groups128;
        d.N += w.N; d.groups64 += w.groups64; d.groups128 += w.groups128; d.payload += w.payload;
    }
    wide64.units = d.groups64;
    wide128.units = d.groups128;
    if (path == PATCH_PATH_AUTO) {
        const AutoChoice c = auto_choice(a, d, set.N, variant == 0 && split_k == 0);
        path = c.path;
        if (c.one_pass) {
            launch_batch_set(a, wide128, 0, (int)M, c.pass.chunks, s);
            HIP_TRY(hipGetLastError());
            return PATCH_OK;
        }
    }
    // (a split asked for is that of one launch per weight, but for the kernel with 128 features, whose chunks cover the set)
    if (split_k != 0 && !(path == PATCH_PATH_DECODE && variant == 7)) { a.ws = nullptr; a.ws_bytes = 0; }
    if (path == PATCH_PATH_PREFILL && (variant == 0 || variant == 3) && split_k <= 1 && prefill_wreg_supports(a)) {
        // one launch over the feature blocks of all weights (with a workspace and few blocks: K in slices over the
        // whole set, see launch_prefill_wreg_set)
        int blocks = 0;
        WeightSet set = {};
        for (int i = 0; i < count; ++i) {
            set.payload[i] = P[i]->d_payload;
            set.table[i] = P[i]->d_table;
            set.Y[i] = static_cast<float*>(Y[i]);
            set.N[i] = P[i]->N;
            set.first[i] = blocks;
            blocks += (int)((P[i]->N + 255) / 256);
        }
        set.count = count;
        set.units = blocks;
        const int split128 = variant == 0 && split_k == 0 ? prefill_r128_split(a, set.N, count) : 0;
        if (split128) launch_prefill_r128(a, set, split128, s);
        else launch_prefill_wreg_set(a, set, s);
        HIP_TRY(hipGetLastError());
        return PATCH_OK;
    }
    if (path == PATCH_PATH_PREFILL) {
        patch_gemm_opts o = {path, split_k, variant, opts ? opts->workspace : nullptr, opts ? opts->workspace_bytes : 0, a.ybf16};
        for (int i = 0; i < count; ++i) {
            const patch_status st = patch_gemm_ex(X, M, P[i], Y[i], stream, &o);
            if (st != PATCH_OK) return st;
        }
        return PATCH_OK;
    }
    for (int64_t m0 = 0; m0 < M; m0 += (variant == 7 ? kBatchRows : kDecodeRows)) {
        const int rows = (int)((M - m0 < (variant == 7 ? kBatchRows : kDecodeRows)) ? M - m0 : (variant == 7 ? kBatchRows : kDecodeRows));
        DecodePlan plan = {0, 1, 0.0};
        if (variant == 4) plan.kernel = 1;
        else if (variant == 7) plan = batch_plan(a, d, rows, split_k);
        else if (variant == 0 && split_k == 0) plan = decode_plan(a, d, rows);
        if (plan.kernel == 2) launch_batch_set(a, wide128, m0, rows, plan.chunks, s);
        else if (plan.kernel == 1) launch_mid_set(a, wide64, m0, rows, 1, s, plan.deal);
        else launch_decode_set(a, set, m0, rows, split_k, variant, s, plan.deal);
    }
    HIP_TRY(hipGetLastError());
    return PATCH_OK;
}

patch_status patch_gemm(const void* X, int64_t M, const patch_packed* P, void* Y, void* stream) {
    return patch_gemm_ex(X, M, P, Y, stream, nullptr);
}

patch_status patch_gemm_static(const void* X, int64_t M, const patch_packed* P, void* Y, void* stream) {
    if (!X || !P || !Y || M < 0) return PATCH_ERR_ARG;
    // (a rule of its own beside what the launch below uses: the calls that were refused or accepted once stay so)
    const size_t need = workspace_need(M, P, nullptr, true);
    if (need > kStaticScratchBytes) return PATCH_ERR_SIZE;
    void* ws = nullptr;
    const patch_status st = static_scratch(&ws);
    if (st != PATCH_OK) return st;
    const patch_gemm_opts o = {PATCH_PATH_AUTO, 0, 0, ws, kStaticScratchBytes, 0};
    return patch_gemm_ex(X, M, P, Y, stream, &o);
}

patch_status patch_unpack(const patch_packed* P, void* W_out, void* stream) {
    if (!P || !W_out || !aligned16(W_out)) return PATCH_ERR_ARG;
    launch_unpack(P->d_payload, P->d_table, P->Tn * P->Tk, P->Tk, P->tile, P->K, static_cast<uint16_t*>(W_out),
                  static_cast<hipStream_t>(stream));
    HIP_TRY(hipGetLastError());
    return PATCH_OK;
}

size_t patch_packed_bytes(const patch_packed* P) { return P ? P->payload_bytes : 0; }
size_t patch_table_bytes(const patch_packed* P) { return P ? (P->table.size() + P->pairs.size()) * sizeof(uint32_t) : 0; }

patch_status patch_packed_dims(const patch_packed* P, int64_t* N, int64_t* K, int* tile, int64_t* n_sparse_tiles) {
    if (!P) return PATCH_ERR_ARG;
    if (N) *N = P->N;
    if (K) *K = P->K;
    if (tile) *tile = P->tile;
    if (n_sparse_tiles) *n_sparse_tiles = P->n_sparse;
    return PATCH_OK;
}

patch_status patch_packed_tile_map(const patch_packed* P, uint8_t* tile_map, size_t bytes) {
    if (!P || !tile_map) return PATCH_ERR_ARG;
    if (bytes < P->tile_map.size()) return PATCH_ERR_SIZE;
    memcpy(tile_map, P->tile_map.data(), P->tile_map.size());
    return PATCH_OK;
}

patch_status patch_packed_row_order(const patch_packed* P, int32_t* order, size_t cap, size_t* count) {
    if (!P || !order || !count) return PATCH_ERR_ARG;
    if (cap < P->pairs.size()) return PATCH_ERR_SIZE;
    if (!P->pairs.empty()) memcpy(order, P->pairs.data(), P->pairs.size() * sizeof(int32_t));
    *count = P->pairs.size();
    return PATCH_OK;
}

patch_status patch_canonical_sizes(const patch_packed* P, size_t* vals_bytes, size_t* meta_bytes) {
    if (!P) return PATCH_ERR_ARG;
    const size_t t2 = (size_t)P->tile * P->tile;
    const size_t n_dense = P->tile_map.size() - (size_t)P->n_sparse;
    if (vals_bytes) *vals_bytes = 2 * (n_dense * t2 + (size_t)P->n_sparse * t2 / 2);
    if (meta_bytes) *meta_bytes = (size_t)P->n_sparse * t2 / 8;
    return PATCH_OK;
}

// Host-side re-ordering of the device layout into the canonical order (test hook; not a hot path).
patch_status patch_export_canonical(const patch_packed* P, void* vals, size_t vals_bytes, void* meta, size_t meta_bytes) {
    if (!P || !vals || (!meta && P->n_sparse)) return PATCH_ERR_ARG;
    size_t need_v = 0, need_m = 0;
    patch_canonical_sizes(P, &need_v, &need_m);
    if (vals_bytes < need_v || meta_bytes < need_m) return PATCH_ERR_SIZE;
    std::vector<uint8_t> host;
    try { host.resize(P->payload_bytes); } catch (...) { return PATCH_ERR_ALLOC; }
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(host.data(), P->d_payload, P->payload_bytes, hipMemcpyDeviceToHost));
    const int t = P->tile, KPT = t / kStepCols;
    uint16_t* v = static_cast<uint16_t*>(vals);
    uint8_t* mt = static_cast<uint8_t*>(meta);
    if (need_m) memset(mt, 0, need_m);
    size_t vi = 0, nib = 0;
    for (size_t ti = 0; ti < P->table.size(); ++ti) {
        const uint32_t e = P->table[ti];
        const uint8_t* base = host.data() + entry_offset(e);
        for (int r = 0; r < t; ++r) {
            const int s = r / 16, i = r % 16;
            if (!entry_sparse(e)) {
                for (int c = 0; c < t; ++c) {
                    const int j = c / 64, h = (c % 64) / 32, q = (c % 32) / 8, el = c % 8;
                    const size_t byte = (size_t)(((s * KPT + j) * 2 + h) * 64 + (16 * q + i)) * 16 + 2 * el;
                    uint16_t x;
                    memcpy(&x, base + byte, 2);
                    v[vi++] = x;
                }
            } else {
                for (int g = 0; g < t / 4; ++g) {
                    const int c = 4 * g, j = c / 64, qa = (c % 64) / 16, gl = (c % 16) / 4;
                    const int lane = 16 * qa + i;
                    const size_t byte = (size_t)((s * KPT + j) * 64 + lane) * 16 + 4 * gl;
                    uint16_t x[2];
                    memcpy(x, base + byte, 4);
                    v[vi++] = x[0];
                    v[vi++] = x[1];
                    uint16_t idx;
                    memcpy(&idx, base + sparse_vals_bytes(t) + (size_t)((s * 64 + lane) * KPT + j) * 2, 2);
                    const uint8_t nibble = (uint8_t)((idx >> (4 * gl)) & 0xF);
                    mt[nib >> 1] |= (uint8_t)(nibble << (4 * (nib & 1)));
                    ++nib;
                }
            }
        }
    }
    return PATCH_OK;
}

}  // extern "C"
