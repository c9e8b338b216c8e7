// C ABI of the FC-layer GEMM library (see include/axonn_linear.h for the contract).
// Host side: argument checks, kernel-variant selection, launch.  No device memory is allocated
// anywhere in this file, and the GEMM entry points never synchronise: split-K kernels exchange their
// partial tiles through memory the caller registered (axonn_linear_set_workspace, which clears the
// flag words synchronously) or, for the one entry point made for callers that cannot allocate,
// through a file-scope device array.
#include "../../include/axonn_linear.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>

#include <vector>

#include "kernels.hpp"
#include "gemm_mfma16.hpp"       // tile configurations only: the kernels are instantiated in kernels_*.hip
#include "gemm_mfma16_k64.hpp"
#include "gemm_mfma16_k64p.hpp"
#include "gemm_edge.hpp"
#include "comm_model.hpp"
#include "transpose.hpp"

namespace axonn {

// ------------------------------------------------------------------------------------------
// Variant 0: guarded kernel, one thread per output element, any M, N, K >= 0.
// fp32 accumulation in ascending k, one RNE rounding at the store.
// ------------------------------------------------------------------------------------------
template <int LAYOUT>
__global__ __launch_bounds__(256) void gemm_naive_kernel(const uint16_t* __restrict__ A,
                                                         const uint16_t* __restrict__ B,
                                                         uint16_t* __restrict__ C, int64_t M,
                                                         int64_t N, int64_t K) {
    // 16 x 16 output blocks, numbered row-major, dealt out to the workgroups of a 1-D grid in turn
    const int64_t blocks_n = (N + 15) / 16, blocks = ((M + 15) / 16) * blocks_n;
    for (int64_t blk = blockIdx.x; blk < blocks; blk += gridDim.x) {
        const int64_t j = (blk % blocks_n) * 16 + (threadIdx.x & 15);
        const int64_t i = (blk / blocks_n) * 16 + (threadIdx.x >> 4);
        if (i >= M || j >= N) continue;
        float acc = 0.f;
        for (int64_t k = 0; k < K; ++k) {
            const uint16_t a = (LAYOUT == AXONN_TN) ? A[k * M + i] : A[i * K + k];
            const uint16_t b = (LAYOUT == AXONN_NT) ? B[j * K + k] : B[k * N + j];
            acc += __builtin_bit_cast(float, (uint32_t)a << 16) * __builtin_bit_cast(float, (uint32_t)b << 16);
        }
        C[i * N + j] = (uint16_t)(pack2_bf16(acc, 0.f) & 0xFFFFu);
    }
}

// ------------------------------------------------------------------------------------------
// Variant table
// ------------------------------------------------------------------------------------------
struct Variant {
    const char* name;
    int bm, bn, threads, lds_bytes, min_k;  // bm == 0: the naive kernel; min_k per K range
    int kstep;                       // K (per range) must be a multiple of this
    int splits;                      // K ranges per tile (1: no split-K)
    bool k64;                        // the kernel with 64-k LDS stages
    // Throughput with every CU busy, per layout (NN, NT, TN), N(0,1) data, in units of about 1200 TFLOP/s.
    // `python -m paper_2502_08145_amd.sweeps variant_eff [--hot]` times every variant without split-K on
    // full-chip shapes and prints such a table.  The numbers below were taken that way as each kernel came
    // in; a re-measurement of all of them at once, with operands from HBM and with operands in cache,
    // gave tables whose plans ran the benchmark step and the model-zoo sweep 0.5-1 % slower (the small
    // tiles are picked for small outputs, which stay in cache, the large ones for large outputs, which
    // do not: neither condition alone describes both), so these stand.
    double eff[3];
    tile_kernel_t fn[3];             // per layout
    // Microseconds per 64 k of a full round of workgroups, per layout, operands in cache (block_us); 0: not used there.
    double us64[3] = {0.0, 0.0, 0.0};
    tile_kernel_t fn_tail[3] = {nullptr, nullptr, nullptr};   // for a K that is no multiple of 64
    bool edge = false;               // the guarded MFMA kernel: any shape, launched through edge_kernel_launch
    int resident = 0;                // > 0: a grid of at most this many workgroups walks the tiles (one per compute unit)
    bool group = false;              // the eight-wave kernel (gemm_tile_kernel_k64g)
    bool group_model = false;        // ... and its time model (block_us)
};

// Kernel families: the 64-k-stage kernel (256 x 256, eight waves: the default wherever the output has
// whole large tiles), the 32-k ring (the same tile for NT at very long K and TN with four and more K
// ranges; the smaller tiles with split-K), the eight-wave kernel (128 x 128 and half tiles without split-K), the guarded kernel.
// Split-K variants of one tile share one kernel (the number of K ranges is a run-time argument).  128 x 128 tiles with split-K
// are the ring's for NN and TN and the four-wave 64-k kernel's for NT, under one name.
static std::vector<Variant> make_variants() {
    std::vector<Variant> v;
    v.push_back({"naive", 0, 0, 256, 0, 0, 1, 1, false, {0, 0, 0}, {nullptr, nullptr, nullptr}});
    auto ring = [&](const char* name, int bm, int bn, int wn, int splits, int lds, int min_k, double nn, double nt, double tn) {
        Variant x{name, bm, bn, 128 * wn, lds, min_k, 2 * KB, splits, false, {nn, nt, tn}, {nullptr, nullptr, nullptr}};
        for (int l = 0; l < 3; ++l)
            x.fn[l] = (bm == 256 && bn == 256)              ? ring_kernel_large(splits > 1, l)
                      : (bm == 128 && bn == 128 && l == AXONN_NT) ? k64_kernel_half(bm, bn, l)
                                                              : ring_kernel_small(bm, bn, l);
        v.push_back(x);
    };
    auto group = [&](const char* name, int bm, int bn, int min_k, bool k64, double nn, double nt, double tn) {
        Variant x{name, bm, bn, 512, group_lds_bytes(bm, bn, 1), min_k, TileCfgK64::KS, 1, k64, {nn, nt, tn}, {nullptr, nullptr, nullptr}};
        x.group = x.group_model = true;
        for (int l = 0; l < 3; ++l)
            if (!k64 || l == AXONN_NT) {
                x.fn[l] = group_kernel(bm, bn, 1, l, false);
                x.fn_tail[l] = group_kernel(bm, bn, 1, l, true);
            }
        v.push_back(x);
    };
    auto k64 = [&](const char* name, int splits) {
        Variant x{name, 256, 256, 512, k64_lds_bytes(256, 256, 1), TileCfgK64::MIN_K, TileCfgK64::KS, splits, true,
                  {1.17, 1.17, 1.15}, {nullptr, nullptr, nullptr}};
        for (int l = 0; l < 3; ++l) x.fn[l] = k64_kernel(splits > 1, l);
        v.push_back(x);
    };
    using L = TileCfg16<256, 256, 2, 4>;
    ring("mfma16_256x256_w8", 256, 256, 4, 1, L::LDS_BYTES, L::MIN_K, 1.13, 1.06, 1.12);
    static const char* const ring_sk[] = {"mfma16_256x256_w8_sk2", "mfma16_256x256_w8_sk3", "mfma16_256x256_w8_sk4", "mfma16_256x256_w8_sk5",
                                          "mfma16_256x256_w8_sk6", "mfma16_256x256_w8_sk7", "mfma16_256x256_w8_sk8"};
    for (int sp = 2; sp <= 8; ++sp) ring(ring_sk[sp - 2], 256, 256, 4, sp, L::LDS_BYTES, L::MIN_K, 1.13, 1.06, 1.12);
    group("mfma16_256x128", 256, 128, TileCfg16<256, 128, 2, 2>::MIN_K, false, 0.86, 0.78, 0.91);
    // The variant that plans of 128 large tiles carry, in NN above all.  Its blocks, and plans with strips that have one, are priced with
    // the ring's figures (us64): near a tie they then go to another tile or to one launch (settle_parts, make_plan).  Priced as the
    // eight-wave kernel, 85 sampled ragged products that changed to strips took 1.05 times as long (1.25 the worst), 8064 x 2944 x 12800 NN
    // 495 us for 428.
    group("mfma16_128x256", 128, 256, TileCfg16<128, 256, 2, 2>::MIN_K, false, 0.95, 0.74, 0.92);
    v.back().group_model = false;
    std::fill(v.back().fn_tail, v.back().fn_tail + 3, nullptr);
    group("mfma16_128x256_w8", 128, 256, TileCfg16<128, 256, 2, 4>::MIN_K, false, 0.93, 0.72, 0.97);
    using S = TileCfg16<128, 128, 2, 2>;
    group("mfma16_128x128", 128, 128, S::MIN_K, false, 0.85, 0.72, 0.90);
    // with split-K NT runs the 64-k kernel with three buffers on this tile, under the same variants
    static_assert(S::LDS_BYTES >= k64_lds_bytes(128, 128, 3) && S::MIN_K >= TileCfgK64::MIN_K, "one LDS size and shortest K for both kernels");
    ring("mfma16_128x128_sk2", 128, 128, 2, 2, S::LDS_BYTES, S::MIN_K, 0.85, 0.72, 0.90);
    ring("mfma16_128x128_sk4", 128, 128, 2, 4, S::LDS_BYTES, S::MIN_K, 0.85, 0.72, 0.90);
    k64("mfma16k64_256x256_w8", 1);
    {
        Variant x{"mfma16k64p_256x256_w8", 256, 256, 512, TileCfgK64P::LDS_BYTES, TileCfgK64::MIN_K, TileCfgK64::KS, 1, true,
                  {1.20, 1.13, 1.17}, {nullptr, nullptr, nullptr}};
        for (int l = 0; l < 3; ++l) x.fn[l] = k64p_kernel(l);
        x.resident = TileCfgK64P::MAX_WORKGROUPS;
        v.push_back(x);
    }
    // half tiles of two K-contiguous operands (eff from 2048 x 4096 x 4096 and 4096^3 against the ring's half tiles)
    auto k64h = [&](const char* name, int bm, int bn, int splits, double nt) {
        Variant x{name, bm, bn, 256, k64_lds_bytes(bm, bn, 3), TileCfgK64::MIN_K, TileCfgK64::KS, splits, true,
                  {0.0, nt, 0.0}, {nullptr, nullptr, nullptr}};
        for (int l = 0; l < 3; ++l) x.fn[l] = k64_kernel_half(bm, bn, l);
        v.push_back(x);
    };
    group("mfma16k64_256x128", 256, 128, TileCfgK64::MIN_K, true, 0.0, 0.95, 0.0);
    group("mfma16k64_128x256", 128, 256, TileCfgK64::MIN_K, true, 0.0, 0.94, 0.0);
    // split-K on the half tiles, for outputs that are narrow in one direction (2048 x 1152, 640 x 15360 ...) over a
    // long K: the 64-k kernel for NT, the 32-k ring for NN and TN
    // (two and three ranges only: with four and more the reader's turn at the slots costs more than the large
    // tile's split-K or 128 x 128 tiles do on the same outputs)
    static const char* const h1_sk[] = {"mfma16k64_256x128_sk2", "mfma16k64_256x128_sk3"};
    static const char* const h2_sk[] = {"mfma16k64_128x256_sk2", "mfma16k64_128x256_sk3"};
    static const char* const r1_sk[] = {"mfma16_256x128_sk2", "mfma16_256x128_sk3"};
    static const char* const r2_sk[] = {"mfma16_128x256_sk2", "mfma16_128x256_sk3"};
    for (int sp = 2; sp <= 3; ++sp) {
        k64h(h1_sk[sp - 2], 256, 128, sp, 0.85);
        k64h(h2_sk[sp - 2], 128, 256, sp, 0.84);
        ring(r1_sk[sp - 2], 256, 128, 2, sp, TileCfg16<256, 128, 2, 2>::LDS_BYTES, TileCfg16<256, 128, 2, 2>::MIN_K, 0.80, 0.70, 0.84);
        ring(r2_sk[sp - 2], 128, 256, 2, sp, TileCfg16<128, 256, 2, 2>::LDS_BYTES, TileCfg16<128, 256, 2, 2>::MIN_K, 0.80, 0.68, 0.82);
    }
    static const char* const k64_sk[] = {"mfma16k64_256x256_w8_sk2", "mfma16k64_256x256_w8_sk3", "mfma16k64_256x256_w8_sk4", "mfma16k64_256x256_w8_sk5",
                                         "mfma16k64_256x256_w8_sk6", "mfma16k64_256x256_w8_sk7", "mfma16k64_256x256_w8_sk8"};
    for (int sp = 2; sp <= 8; ++sp) k64(k64_sk[sp - 2], sp);
    // us64: fitted over 36 000 sampled products (residual 3-4 %, 128 x 128 tiles 7-8 %).  The eight-wave kernel's are those of
    // the kernels that had its tiles when the rule for the scratch area was made (Figures::Area); nothing else reads them.
    static const struct { const char* name; double us64[3]; } measured[] = {
        {"mfma16_128x128", {0.530, 0.525, 0.557}},       {"mfma16_128x256", {0.927, 0.887, 0.950}},
        {"mfma16_128x256_w8", {0.773, 0.818, 0.852}},    {"mfma16_256x128", {0.885, 0.888, 0.951}},
        {"mfma16k64_128x256", {0.0, 0.817, 0.0}},        {"mfma16k64_256x128", {0.0, 0.819, 0.0}},
        {"mfma16k64_256x256_w8", {1.284, 1.219, 1.263}},
    };
    for (Variant& x : v)
        for (const auto& q : measured)
            // a split-K variant's name is the plain one's and "_sk<ranges>"
            if (std::strncmp(x.name, q.name, std::strlen(q.name)) == 0 && (x.splits > 1) == (std::strstr(x.name, "_sk") == x.name + std::strlen(q.name)) &&
                (x.splits > 1 || std::strlen(x.name) == std::strlen(q.name))) {
                std::copy(q.us64, q.us64 + 3, x.us64);
                for (int l = 0; l < 3 && x.splits == 1 && x.bm * x.bn == 256 * 256; ++l) x.fn_tail[l] = k64_kernel(false, l, true);
            }
    // guarded MFMA kernel: any shape; a plan's blocks under this name run on what guarded_choice takes for them
    Variant e{"mfma16_edge_128x128", EdgeCfg::BM, EdgeCfg::BN, EdgeCfg::NT, EdgeCfg::LDS_BYTES, 1, 1, 1, false, {0, 0, 0}, {nullptr, nullptr, nullptr}};
    e.edge = true;
    v.push_back(e);
    return v;
}
static const std::vector<Variant>& variants() {
    static const std::vector<Variant> table = make_variants();
    return table;
}
static int num_variants() { return (int)variants().size(); }
static int edge_variant() { return num_variants() - 1; }
static bool is_guarded(int v) { return variants()[v].bm == 0 || variants()[v].edge; }

// Split-K scratch: one area per device.  Layout: kFlagBytes of flags (one 32-bit flag per slot, the
// time-out counter in the last word), then slots of one 256x256 fp32 tile each.  The area is the
// caller's (axonn_linear_set_workspace); without one the three GEMM entry points run the kernels that
// need none.  The library itself allocates nothing.
constexpr int kScratchSlots = 256;                          // the most any variant is allowed to need
constexpr size_t kSlotBytes = 256 * 256 * sizeof(float);
constexpr size_t kFlagBytes = 4096;                         // 1023 flags + the counter
constexpr int64_t kMaxFlags = kFlagBytes / sizeof(uint32_t) - 1;
constexpr int kMaxDevices = 64;
struct Scratch {
    float* partials = nullptr;
    uint32_t* flags = nullptr;
    size_t partial_bytes = 0;       // capacity behind `partials`
    uint32_t* timeouts() const { return flags + kFlagBytes / sizeof(uint32_t) - 1; }
};
static Scratch g_scratch[kMaxDevices];
static std::mutex g_scratch_mutex;
static std::atomic<uint32_t> g_epoch{0};
static std::atomic<int> g_split_k_enabled{1};

static Scratch carve(void* p, size_t bytes) {
    Scratch sc;
    sc.flags = static_cast<uint32_t*>(p);
    sc.partials = reinterpret_cast<float*>(static_cast<char*>(p) + kFlagBytes);
    sc.partial_bytes = bytes - kFlagBytes;
    return sc;
}

// The current device's registered area (by value: a later set_workspace does not disturb a launch
// being prepared) if it has room for `bytes_needed` bytes of partial tiles; else .partials == nullptr.
static Scratch registered_scratch(size_t bytes_needed) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return Scratch{};
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    const Scratch& sc = g_scratch[dev];
    return (sc.partials && sc.partial_bytes >= bytes_needed) ? sc : Scratch{};
}

// The scratch area of the entry point for callers that cannot allocate: a device array of fixed size
// that every GPU the library runs on holds from the moment the code object is loaded until the
// process ends (zero-filled at load).  In host code the array's NAME is only a handle for
// hipGetSymbolAddress; the address kernels and copies may use is looked up once per device, with that
// device current, and kept in g_static_ptr.
constexpr int kStaticSlots = 128;                           // 32 MiB of partial tiles
constexpr size_t kStaticBytes = kFlagBytes + kStaticSlots * kSlotBytes;
static __device__ __align__(256) unsigned char g_static_scratch[kStaticBytes];
static unsigned char* g_static_ptr[kMaxDevices];
static std::mutex g_static_mutex;

// The current device's copy of the static area; .partials == nullptr if the look-up failed.
static Scratch static_scratch() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return Scratch{};
    }
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return Scratch{};
        }
        g_static_ptr[dev] = static_cast<unsigned char*>(p);
    }
    return carve(g_static_ptr[dev], kStaticBytes);
}

static std::atomic<int> g_forced{-1};
static std::once_flag g_attr_once[kMaxDevices];   // the LDS limits are a per-device property of a kernel

// per-lane address offsets are 32 bits: up to 16 rows of a K-contiguous operand, 4 (64-k kernel: 36)
// k-rows of an MN-contiguous one, plus the K window of a K-contiguous one
constexpr int64_t kMaxTileDim = (int64_t)1 << 24;

static bool variant_supports(int v, int64_t M, int64_t N, int64_t K, int layout) {
    if (v < 0 || v >= num_variants() || layout < 0 || layout > 2) return false;
    const Variant& var = variants()[v];
    if (var.bm == 0) return true;
    if (M <= 0 || N <= 0 || K <= 0) return false;
    if (var.edge) return ((M + var.bm - 1) / var.bm) * ((N + var.bn - 1) / var.bn) < ((int64_t)1 << 31);
    if (!var.fn[layout]) return false;   // a kernel for one layout only
    if (M > kMaxTileDim || N > kMaxTileDim || K > kMaxTileDim) return false;
    if (M % var.bm != 0 || N % var.bn != 0 || K % (var.kstep * var.splits) != 0 || K / var.splits < var.min_k) return false;
    if (var.splits == 1) return true;
    // scratch: one flag and one fp32 tile per (tile, extra K range)
    const int64_t slots = (M / var.bm) * (N / var.bn) * (var.splits - 1);
    return slots <= kMaxFlags && slots * var.bm * var.bn * (int64_t)sizeof(float) <= (int64_t)(kScratchSlots * kSlotBytes);
}

// Tile-shape choice.  MI355X has 256 compute units; a partly filled last round of tiles costs a
// whole tile time, and a smaller tile moves more operand bytes per flop.  Pick the variant with the
// smallest modelled time:
//     rounds x tile area x (K per workgroup + fixed cost) / efficiency
// where the efficiencies are throughputs measured on MI355X with every CU busy (N(0,1) data, see
// Variant::eff), and the fixed cost (pipeline fill, epilogue,
// for split-K also the exchange of fp32 partial tiles) is expressed in units of k.
// K-contiguous operands are the dearer ones to stage (64-byte row segments per load), which is
// why NN likes a short A tile (128x256) and NT gains least from any of the smaller tiles.
// Split-K turns an output of at most 128 tiles of 256x256 into a full round of the large tile.
static double model_time(int v, int64_t M, int64_t N, int64_t K, int layout, bool allow_split) {
    constexpr double kFixedK = 128.0;
    const Variant& var = variants()[v];
    if (!variant_supports(v, M, N, K, layout) || (var.splits > 1 && !allow_split) || var.eff[layout] <= 0.0) return -1.0;
    // Long K: without split-K the 64-k kernels lead the 32-k ring in every mode (8192 x 8192 x 32768 and
    // x 49152: NN and TN by 1-5 %, NT, since its A panel is triple-buffered, by 9-10 %).  With split-K
    // they lead in NN and NT at any K tried (2048 x 2048 x 65536 in four ranges: +5 % and +11 %;
    // 1024 x 2048 x 131072 in eight: +3 % and +13 %), in TN the ring is level or up to 8 % ahead above
    // K = 32768.
    if (var.k64 && var.splits > 1 && layout == AXONN_TN && K > 32768) return -1.0;
    // The resident-workgroup form of the 64-k kernel: measured against one workgroup per tile in the
    // benchmark's sequence, 1.3-1.9 % less time for the TN products of three and four tiles per compute
    // unit, +-1 % for NN, 1.6 % MORE for NT with two tiles and 2.5 % more with a single tile.
    // What it saves is per tile: at K = 16384 and 32768 it measures 2.5-5 % behind one workgroup per tile.
    // NN at K = 2048 (4096 x 16384 x 2048, four tiles per compute unit): 226 -> 220 us.
    if (var.resident > 0 && !((layout == AXONN_TN || (layout == AXONN_NN && K <= 2048)) && (M / var.bm) * (N / var.bn) >= 3 * var.resident && K <= 8192)) return -1.0;
    const int64_t wgs = (M / var.bm) * (N / var.bn) * var.splits;
    // Every CU works through ceil(wgs / 256) workgroups (two small tiles resident on one CU run
    // side by side at half speed each, which comes to the same).  A last round that fills only
    // a fraction f of the CUs runs faster than a full one (the busy CUs get the idle ones'
    // power and bandwidth): measured about 0.6 + 0.4 f of a full round (0.61 at 4 workgroups,
    // 0.78 at 128, 0.87 at 144).
    const int64_t full = wgs / 256, rest = wgs % 256;
    // readers and writers of a tile should run side by side: one round of large tiles, two of small ones
    if (var.splits > 1 && wgs > (var.bm * var.bn <= 128 * 128 ? 512 : 256)) return -1.0;
    const double rounds = (double)full + (rest ? 0.6 + 0.4 * (double)rest / 256.0 : 0.0);
    // the exchange of a small tile is latency: the reader takes the partial tiles one after the
    // other once the writers are done, and it grows with the number of tiles in flight
    // (measured: 4 us + 0.055 us per tile for two K ranges, 7 us + 0.17 us per tile for four)
    const double tiles = (double)((M / var.bm) * (N / var.bn));
    const double fixed_small = var.splits == 2 ? 700.0 + 8.0 * tiles : 1300.0 + 25.0 * tiles;
    // large tiles: the partial tiles travel through HBM, (splits - 1) x 256 KB per tile written and
    // read back at 4-5 TB/s (0.1 us, or 4 units of k, per slot), and the reader of a tile takes its
    // slots one after the other at one CU's rate (2.5 us, 100 units, per slot)
    // (half tiles: half the bytes per slot in flight; what the reader pays per slot is mostly latency)
    const bool half_tile = var.bm * var.bn < 256 * 256;
    const double fixed_large = 4.0 * tiles * (var.splits - 1) * (var.bm * var.bn) / 65536.0 + (half_tile ? 160.0 : 100.0) * (var.splits - 1);
    const double k_cost = (double)(K / var.splits) + kFixedK +
                          (var.splits == 1 ? 0.0 : var.bm * var.bn <= 128 * 128 ? fixed_small : fixed_large);
    double e = var.eff[layout];
    // the 64-k kernel leads the 32-k ring in TN by 2-4 % in one range and in two (six clusters of
    // transposing reads, streamed epilogue); with four ranges and more it measured 2-4 % behind
    if (layout == AXONN_TN && var.k64 && var.splits >= 4) e *= 0.94;
    return rounds * var.bm * var.bn * k_cost / e;
}

// model_time's units to the microsecond: a 256 x 256 tile over K = 4096 is 2.7e8 and takes about 100 us
constexpr double kUnitsPerUs = 2.6e6;

// The guarded MFMA kernel (gemm_edge_kernel) alone, in microseconds: steps of 128 k, dearer nearly in proportion as
// workgroups come to share the compute units (least squares over 15 000 sampled products each of aligned and of
// misaligned rows, residual 6 % and 23 %; aligned rows also over 900 outputs of up to 500 MB, 10 %, where
// proportion was 12-15 % too much).
static double edge_us(int64_t m, int64_t n, int64_t K, bool rows_aligned) {
    const double wgs = (double)(((m + EdgeCfg::BM - 1) / EdgeCfg::BM) * ((n + EdgeCfg::BN - 1) / EdgeCfg::BN));
    const double steps = (double)((K + EdgeCfg::BK - 1) / EdgeCfg::BK);
    return rows_aligned ? 3.0 + (1.8 * steps + 2.6) * std::pow(1.0 + (wgs / 287.0) * (wgs / 287.0), 0.47)
                        : 3.0 + (2.0 * steps + 5.0) * std::sqrt(1.0 + (wgs / 292.0) * (wgs / 292.0));
}

// Whose figures a modelled time is made of.
// Area: the ones that decide which products exchange partial tiles through the scratch area.  That set is part of the
// interface -- other products can overlap on several streams, and the static entry never refuses them -- so it does
// not follow the kernels: these figures stay, and compare whole tiles and split-K, and the wave-K kernel, in one unit (operands
// in cache).  While it did follow the refitted ones, which are the mean of operands in cache and from memory but for split-K,
// 1 % of sampled ragged products went from one launch without scratch to whole tiles with split-K and strips: thirty of those, in
// one launch and so, 0.88 times as fast (6984 x 6056 x 9856 NN 615 us and 762).
enum class Figures { Current, Area };

// How a block of the output is computed where it is not simply the tile variant of its part.
struct BlockChoice {
    int tile = -1;           // >= 0: this tile variant, its last tiles moved back to the block's edge (TileGrid)
    GroupChoice group{};     // else, .tile >= 0: one of the eight-wave kernel's small tiles
    WaveKChoice wavek{};     // else, .tile >= 0: the wave-K kernel
    GroupSplitChoice split{};     // else, .tile >= 0: the eight-wave kernel in K ranges, where the scratch area has room; else what the part's variant says
    int lead_m = 0, lead_n = 0;   // rows and columns before the block that the launch covers as well
    double us = 0.0;         // modelled time
};

// Where the rows of the output do not start on 128-byte lines, a tile's stores end in lines that two workgroups write a
// part of.  That costs a round of 256 x 256 tiles 6.4 us (but for the first half round), one of half tiles 1.4, one of
// 128 x 128 tiles 0.6 from 8 rounds on; less where the rows start on 32 or 64 bytes.  Medians of 800 sampled products,
// each measured on every tile; without it the model was short by up to 1.7 times for outputs of 240 MB and more.
static double shared_lines_us(const Variant& x, int64_t m, int64_t n, int64_t ldc) {
    const double share = ldc % 64 == 0 ? 0.0 : ldc % 32 == 0 ? 0.15 : ldc % 16 == 0 ? 0.9 : 1.0;
    const double rounds = (double)(((m + x.bm - 1) / x.bm) * ((n + x.bn - 1) / x.bn) * x.splits) / 256.0;
    const int area = x.bm * x.bn;
    return share * (area <= 128 * 128  ? 0.6 * std::max(0.0, rounds - 8.0)
                    : area < 256 * 256 ? 1.4 * std::max(0.0, rounds - 0.5)
                                       : 6.4 * std::max(0.0, rounds - 0.5));
}

// A tile variant over an m x n block, in microseconds; < 0: it cannot run there, or there is no model of it.
// The eight-wave kernel has a model of its own.  Full rounds of 256 workgroups and 0.76 + 0.24 f of one for a last round that fills a fraction f of the compute
// units; split-K variants also exchange partial tiles, which costs a trip to memory and back per range and
// some of its bandwidth per tile.  Fitted over 36 000 sampled products, residual 3-8 %.
static double block_us(int v, int64_t m, int64_t n, int64_t K, int layout, int64_t lda, int64_t ldb, int64_t ldc, Figures figures = Figures::Current) {
    const Variant& x = variants()[v];
    const bool group = x.group_model && figures == Figures::Current;
    const int64_t k_padded = (K + 63) / 64 * 64;   // every tile kernel takes K 64 at a time
    if ((x.us64[layout] <= 0.0 && !group) || !x.fn[layout] || m < x.bm || n < x.bn || K <= 64) return -1.0;
    if (k_padded / x.splits < x.min_k && !group) return -1.0;   // the eight-wave kernel takes any K
    if (K != k_padded && !x.fn_tail[layout]) return -1.0;
    if (lda % 8 != 0 || ldb % 8 != 0 || ldc % 8 != 0) return -1.0;   // 16-byte direct loads and stores
    if (std::max(std::max(lda, ldb), std::max(ldc, std::max(m, K))) > kMaxTileDim) return -1.0;
    if (group) return group_us(x.bm, x.bn, 1, layout, m, n, K, lda, ldb, ldc);
    const int64_t tiles = ((m + x.bm - 1) / x.bm) * ((n + x.bn - 1) / x.bn), wgs = tiles * x.splits, rest = wgs % 256;
    const double rounds = (double)(wgs / 256) + (rest ? 0.76 + 0.24 * (double)rest / 256.0 : 0.0);
    if (figures == Figures::Current && x.splits == 1 && x.bm * x.bn == 256 * 256) {
        // fitted by itself over 1 500 products of 4 to 600 GFLOP, the mean of operands in cache and from memory (residual 4 %; 8 %
        // with the split forms' figures, which were up to 25 % too much for K of one to four steps)
        static const double step[3] = {1.444, 1.333, 1.411};
        return rounds * ((double)(k_padded / 64) * step[layout] + 6.4) + shared_lines_us(x, m, n, ldc);
    }
    const int area = x.bm * x.bn, more = x.splits - 2;
    const double fixed = area <= 128 * 128 ? 1.9 : area < 256 * 256 ? 3.6 : 5.6;   // per round
    double exchange = 0.0;
    if (x.splits > 1)
        exchange = area <= 128 * 128  ? 4.1 + 1.35 * more + (0.030 + 0.022 * more) * (double)tiles
                   : area < 256 * 256 ? 5.4 + 2.3 * more + (0.044 + 0.030 * more) * (double)tiles
                                      : 6.8 + 2.7 * more + (0.060 + 0.040 * more) * (double)tiles;
    return 3.0 + rounds * ((double)(k_padded / 64 / x.splits) * x.us64[layout] + fixed) + shared_lines_us(x, m, n, ldc) + exchange;
}

// The tile kernel without split-K (overlapping tiles and strips never touch the scratch area) of the smallest modelled time, if
// that is below best.us.
static bool tiles_choice(int64_t m, int64_t n, int64_t K, int layout, int64_t lda, int64_t ldb, int64_t ldc, BlockChoice& best, bool wavek_stays,
                         Figures figures = Figures::Current) {
    bool found = false;
    for (int v = 1; v < edge_variant(); ++v) {
        if (variants()[v].splits > 1) continue;
        const double us = block_us(v, m, n, K, layout, lda, ldb, ldc, figures);
        if (us >= 0.0 && us < best.us) {
            best = BlockChoice{};
            best.tile = v;
            best.us = us;
            found = true;
        }
    }
    if (figures == Figures::Area) return found;
    // The half tiles' model was fitted up to 80 GFLOP.  From 300 on they take 4 to 11 % more of it, beside the 256 x 256 tile's, than there (34
    // products on both; 5768 x 9696 x 12544 NT 1240 us on 128 x 256 tiles, 1091 on 256 x 256).  Near a tie over a long K it is the 256 x 256 tile
    // then: 77 ragged products that this moves run 1.12 times as fast, 82 of K below 6000 would run 1.00 times, 0.98 in NT.  The time
    // stays the half tile's: it is what strips are compared with.
    // Likewise over two steps of K under whole lines of 32 MB of output and more: the models put the smaller tiles up to 1.14 times ahead there,
    // and 36 sampled products ran 0.99 times as fast on them with operands in cache, 0.90 from memory (0.73 the worst, 7808 x 3200 x 128 NN 17.6 us
    // and 24.0); over K of 192 to 512 35 ran 1.10 and 1.03 times.
    const bool long_k = K >= 6000 && 2.0 * (double)m * (double)n * (double)K > 300e9;
    const bool two_steps = K <= 2 * 64 && ldc % 64 == 0 && m * n >= (int64_t)16 << 20;
    bool tie = false;
    if (found && variants()[best.tile].group && (long_k || two_steps))
        for (int v = 1; v < edge_variant(); ++v)
            if (variants()[v].k64 && variants()[v].splits == 1 && variants()[v].bm * variants()[v].bn == 256 * 256) {
                const double us = block_us(v, m, n, K, layout, lda, ldb, ldc);
                if (us >= 0.0 && us < (two_steps ? 1.15 : 1.06) * best.us) {
                    best.tile = v;
                    tie = true;   // with the other tiles of that model as well
                }
            }
    if (lda % 8 != 0 || ldb % 8 != 0 || ldc % 8 != 0 || std::max(std::max(lda, ldb), std::max(ldc, std::max(m, K))) > kMaxTileDim) return found;
    // wavek_stays: near a tie.  Either model is good to 6 %, and where operands come from memory (12 MB and more) its
    // waves, eight chunks of a row in flight between them, suffer less (698 x 968 x 7144 NT: 35 us in cache, 40 from memory; 64 x 64
    // tiles 34 and 51).  In NN by lines (GroupKLines) from smaller operands too (within 12 %: 0.92 to 1.12 times as fast in cache, 0.78 to 0.92 from memory;
    // 506 x 816 x 3112 12.4 us and 13.5, from memory 15.4 and 19.7).
    const GroupChoice g = group_choose(layout, m, n, K, lda, ldb, ldc);
    const bool far = m * K + K * n > (int64_t)6000000 || (layout == AXONN_NN && K % 64 != 0 && K > 2 * kGroupLinesK);
    const double near = tie ? (two_steps ? 1.0 / 1.15 : 1.0 / 1.06) : best.wavek.tile < 0 || !wavek_stays ? 1.0 : far ? 0.88 : 0.96;
    if (g.tile >= 0 && g.us < near * best.us) {
        best = BlockChoice{};
        best.group = g;
        best.us = g.us;
        found = true;
    }
    return found;
}

// The kernel with the smallest modelled time.  The tile kernels win as soon as their tiles fill a good part of the
// chip (1064 x 4168 x 1608 NN: 25 us against 39 for the guarded kernel and 43 for the wave-K one), the wave-K kernel
// wherever the output has few 128 x 128 tiles (by a factor of three and more for a few rows over a long K; it
// loses from some 20 GFLOP on, where its 64 x 64 tiles load twice the bytes: 1930 x 7344 x 1832 NN 123 us against
// 96 for the guarded kernel), the guarded one for large outputs over one or two steps of K (4160 x 11928 x 72 TN: 38 us
// against 53 on 256 x 256 tiles).
// The guarded kernel has to be modelled 9 % shorter below K = 2048: its model is 5 to 11 % short there for rows of two K-contiguous
// operands, the wave-K one 10 to 15 % long for launches of more than some 12 us (taken off up to two chunks of K).  At a tie it was the
// wrong one by up to 1.7 times (8030 x 2081 x 460 NT 41 us on the wave-K kernel, 70 here; 262144 x 128 x 64 TN 18 and 27).  From K = 2048
// on a tie is the guarded kernel's.  1 120 sampled ragged products on all three kernels (K of 8 to 6000, beyond K = 320 the contested
// ones): what is chosen takes 1.005 times the best of the three on average, 1.29 at most; with ties to the guarded kernel 1.018 and 1.76.
static BlockChoice guarded_choice(int64_t m, int64_t n, int64_t K, int layout, int64_t lda, int64_t ldb, int64_t ldc, Figures figures) {
    const bool current = figures == Figures::Current;
    BlockChoice guarded, best;
    guarded.us = edge_us(m, n, K, lda % 8 == 0 && ldb % 8 == 0);
    best.us = (current && K < 2048 ? 1.1 : 0.93) * guarded.us;
    WaveKChoice wk = wavek_choose(layout, m, n, K, lda, ldb, !current);
    if (current && K <= 2 * 64) wk.us -= 0.15 * std::max(0.0, wk.us - 5.0);
    if (wk.tile >= 0 && wk.us < best.us) {
        best.wavek = wk;
        best.us = wk.us;
    }
    if (tiles_choice(m, n, K, layout, lda, ldb, ldc, best, wk.us < 0.93 * guarded.us, figures)) return best;
    return best.wavek.tile < 0 ? guarded : best;
}
// The same for the block at (row0, col0) of the M x N product.  An edge strip of fewer than 16 rows or columns of
// an MN-contiguous operand is too narrow for the wave-K kernel and would take the guarded one, element by element
// (2048 x 8 over K = 4096: 60 us against 12); it takes the 16 last ones instead, some of which the launch over the
// whole tiles, which comes first, has written before.
static BlockChoice guarded_choice(int64_t row0, int64_t col0, int64_t m, int64_t n, int64_t M, int64_t N, int64_t K, int layout,
                                  Figures figures = Figures::Current) {
    const int lead_m = (layout == AXONN_TN && m < 16 && row0 >= 16) ? (int)(16 - m) : 0;
    const int lead_n = (layout != AXONN_NT && n < 16 && col0 >= 16) ? (int)(16 - n) : 0;
    BlockChoice g = guarded_choice(m + lead_m, n + lead_n, K, layout, layout == AXONN_TN ? M : K, layout == AXONN_NT ? K : N, N, figures);
    if (g.tile < 0 && g.group.tile < 0 && g.wavek.tile >= 0) {
        g.lead_m = lead_m;
        g.lead_n = lead_n;
    }
    return g;
}

// The variant with the smallest modelled time for one launch over the whole output (the guarded MFMA
// kernel if no tile shape divides it; 0, the naive kernel, for K = 0); *t_out receives that time.
static int select_variant(int64_t M, int64_t N, int64_t K, int layout, bool allow_split, double* t_out = nullptr) {
    int best = 0;
    double best_t = 0;
    for (int v = 1; v < num_variants(); ++v) {
        const double t = model_time(v, M, N, K, layout, allow_split);
        if (t >= 0.0 && (best == 0 || t < best_t)) {
            best = v;
            best_t = t;
        }
    }
    if (best == 0 && variant_supports(edge_variant(), M, N, K, layout)) {
        best = edge_variant();
        best_t = guarded_choice(0, 0, M, N, M, N, K, layout).us * kUnitsPerUs;
    }
    if (t_out) *t_out = best_t;
    return best;
}

// A product as one launch, or as two launches over disjoint blocks of the output.  An output of,
// say, 384 large tiles keeps the 256 CUs busy for one round and half of them for a second; cut
// into a block of 256 tiles and a block of 128, the second block can run as split-K (or on a
// smaller tile) and fill the chip again.  The cut runs along N (the second block holds the last
// columns) or along M (the last rows); operand and output blocks are addressed through the leading
// dimensions of the whole matrices.
struct Part {
    int variant;
    int64_t m, n, row0, col0;
    BlockChoice how{};   // what the guarded variant runs here; a tile variant may leave the block to the wave-K kernel
};
struct Plan {
    int parts;
    Part part[AXONN_MAX_PLAN_PARTS];
};
static_assert(AXONN_MAX_PLAN_PARTS >= 4, "two launches over whole tiles and two edge strips");

// Whether the whole tiles of a ragged product (mm x nm of its M x N) may use the scratch area.  Products that may
// not can overlap on several streams and are never refused by the static entry, so the set is part of the
// interface: it is fixed by the rates below (a guarded strip's, in microseconds) and does not follow what a ragged
// product's kernels have become since.  Without it 311 of 90 000 sampled products would exchange partial tiles
// through the area that other plans leave alone, twelve of them more than the static area holds.
static bool ragged_may_split(int64_t M, int64_t N, int64_t mm, int64_t nm, int64_t K, int layout) {
    constexpr double kLaunch = 3.0, kStep = 2.0, kSideBySide = 320.0;   // a launch; 128 k; workgroups at that rate
    auto guarded = [&](int64_t m, int64_t n) {
        const double wgs = (double)(((m + 127) / 128) * ((n + 127) / 128));
        return kLaunch + (double)((K + 127) / 128) * kStep * std::max(1.0, wgs / kSideBySide);
    };
    double t = 0.0;
    if (is_guarded(select_variant(mm, nm, K, layout, true, &t))) return false;
    // a strip is a further launch of 8e6 units
    if (nm != N) t += guarded(mm, N - nm) * kUnitsPerUs + 8.0e6;
    if (mm != M) t += guarded(M - mm, N) * kUnitsPerUs + 8.0e6;
    return t < guarded(M, N) * kUnitsPerUs;
}

// Bytes of partial tiles that the variants of a block, or of a plan, exchange.
static size_t split_bytes(const Part& p) {
    const Variant& x = variants()[p.variant];
    return x.splits == 1 ? 0 : (size_t)((p.m / x.bm) * (p.n / x.bn) * (x.splits - 1)) * x.bm * x.bn * sizeof(float);
}

static size_t split_bytes(const Plan& plan) {
    size_t bytes = 0;
    for (int i = 0; i < plan.parts; ++i) bytes = std::max(bytes, split_bytes(plan.part[i]));
    return bytes;   // the launches of a plan run one after the other and share the area
}

// A launch over whole tiles of the M x N product, in microseconds.  The variants without a figure of their own count as
// the 64-k kernel on the same tile: the 32-k ring on the large tile, and the resident workgroups, whose stores overlap
// the next tile's loads (1 to 2 us a round less on 36 products, and 0.6 of what shared lines cost; below K = 384 only
// where there are none).
static double tiles_us(const Part& p, int64_t M, int64_t N, int64_t K, int layout, Figures figures = Figures::Current) {
    const Variant& x = variants()[p.variant];
    const int64_t lda = layout == AXONN_TN ? M : K, ldb = layout == AXONN_NT ? K : N;
    double us = block_us(p.variant, p.m, p.n, K, layout, lda, ldb, N, figures);
    for (int v = 1; us < 0.0 && v < edge_variant(); ++v) {
        const Variant& y = variants()[v];
        if (!y.k64 || y.bm != x.bm || y.bn != x.bn || y.splits != x.splits) continue;
        us = block_us(v, p.m, p.n, K, layout, lda, ldb, N, figures);
        if (us >= 0.0 && x.resident && (N % 64 == 0 || K >= 384)) {
            us -= 1.5 * std::max(0.0, (double)((p.m / x.bm) * (p.n / x.bn)) / x.resident - 1.0);
            us -= 0.4 * shared_lines_us(y, p.m, p.n, N);
        }
    }
    return us < 0.0 ? model_time(p.variant, p.m, p.n, K, layout, true) / kUnitsPerUs : us;
}

static Plan make_plan(int64_t M, int64_t N, int64_t K, int layout, bool allow_split) {
    double t_one = 0;
    Plan plan{1, {{select_variant(M, N, K, layout, allow_split, &t_one), M, N, 0, 0}}};
    if (is_guarded(plan.part[0].variant)) {
        // Ragged output: one launch (guarded_choice: on tile kernels the last tiles overlap their
        // neighbours), or the whole 128 x 128 tiles to the tile kernels (if K suits them) and the last
        // columns and the last rows as strips of their own.  Strips pay where the overlapping tiles would
        // start another round: 2049 x 8192 x 2048 NN is one round of 256 large tiles and a strip of one row
        // (59 us), or 288 tiles in one launch (87 us).
        const int64_t mm = M - M % 128, nm = N - N % 128;
        // the tile kernels move 16 bytes at a time: every row of the operands and of the output, as
        // stored in the whole matrices, has to start on a 16-byte boundary (K is a multiple of 32 here)
        const bool rows_aligned = N % 8 == 0 && (layout != AXONN_TN || M % 8 == 0);
        if (mm > 0 && nm > 0 && (mm != M || nm != N) && rows_aligned) {
            // Up to 640 whole tiles the plans that split took as long as the one launch or longer, which needs no scratch.
            const bool split = allow_split && (mm / 128) * (nm / 128) > 640 && ragged_may_split(M, N, mm, nm, K, layout);
            double t_tiles = 0;
            const int v_tiles = select_variant(mm, nm, K, layout, split, &t_tiles);
            if (!is_guarded(v_tiles)) {
                const Plan inner = make_plan(mm, nm, K, layout, split);
                // One time model on both sides.  Of 1 230 sampled products, each measured in both forms, those whose modelled
                // times are within 5 % of each other took 0.97 (strips modelled shorter) and 1.00 (longer) of the one
                // launch.  Many tiles over a long K keep their strips up to 1.2: the plans of such products
                // (axonn_linear_plan) are relied on as whole tiles and strips, which costs 6-19 % there (2152 x 12296 x
                // 4096 NT 195 us against 179).
                // Below K = 512 the strips have to be clearly shorter: what shared lines cost the whole tiles is the larger
                // part of the time there.
                const double favour = (mm / 128) * (nm / 128) >= 1024 && K >= 4096 ? 1.2 : 1.0;
                auto strips_pay = [&](Figures figures) {
                    double t = 0.0;
                    for (int i = 0; i < inner.parts; ++i) t += tiles_us(inner.part[i], M, N, K, layout, figures);
                    if (nm != N) t += guarded_choice(0, nm, mm, N - nm, M, N, K, layout, figures).us;
                    if (mm != M) t += guarded_choice(mm, 0, M - mm, N, M, N, K, layout, figures).us;
                    if (figures == Figures::Area) return t < favour * guarded_choice(0, 0, M, N, M, N, K, layout, figures).us;
                    return t < (K < 512 ? 0.9 : favour) * t_one / kUnitsPerUs;
                };
                if (strips_pay(Figures::Current) && (split_bytes(inner) == 0 || strips_pay(Figures::Area))) {
                    plan = inner;
                    if (nm != N) plan.part[plan.parts++] = Part{edge_variant(), mm, N - nm, 0, nm};
                    if (mm != M) plan.part[plan.parts++] = Part{edge_variant(), M - mm, N, mm, 0};
                }
            }
        }
        return plan;
    }
    // nothing to gain within half a round of large tiles: split-K and the smaller tiles cover that
    if (M % 128 != 0 || N % 128 != 0 || (M / 128) * (N / 128) <= 4 * 128) return plan;
    // what a second launch costs beyond its own fill and drain (the first one's tail is not
    // overlapped), in the model's units: about 3 us
    constexpr double kSecondLaunch = 8.0e6;
    // a two-launch plan must be clearly better: the model is good to a few per cent
    double best_t = t_one * 0.97;
    auto consider = [&](bool along_n, int64_t rest) {
        const int64_t m1 = along_n ? M : M - rest, n1 = along_n ? N - rest : N;
        const int64_t m2 = along_n ? M : rest, n2 = along_n ? rest : N;
        double t1 = 0, t2 = 0;
        const int v1 = select_variant(m1, n1, K, layout, allow_split, &t1);
        const int v2 = select_variant(m2, n2, K, layout, allow_split, &t2);
        if (is_guarded(v1) || is_guarded(v2) || t1 + t2 + kSecondLaunch >= best_t) return;
        best_t = t1 + t2 + kSecondLaunch;
        plan = Plan{2, {{v1, m1, n1, 0, 0}, {v2, m2, n2, along_n ? 0 : m1, along_n ? n1 : 0}}};
    };
    // second blocks of up to half a round of large tiles, in steps of one tile column / row
    const int64_t step_n = N % 256 == 0 ? 256 : 128, step_m = M % 256 == 0 ? 256 : 128;
    for (int64_t rest = step_n; rest < N && M * rest <= (int64_t)128 * 256 * 256; rest += step_n) consider(true, rest);
    for (int64_t rest = step_m; rest < M && rest * N <= (int64_t)128 * 256 * 256; rest += step_m) consider(false, rest);
    return plan;
}

// Which kernels do the blocks of the guarded variant, and which of a tile variant's blocks are small enough for
// the wave-K kernel: outputs of a few dozen 128 x 128 tiles and fewer, over a K that is long for them (128 x 128 x 8192 NT planned in
// four K ranges 19.4 us, 7.4 on it; 256 x 256 x 8192 21.0 and 8.1).
// A block planned without split-K also goes to whatever other tile kernel without it is modelled faster: the plans are made
// with efficiencies from before the eight-wave kernel, which do not know its smaller tiles.  One planned with split-K
// leaves it for the wave-K kernel only.
// By the scratch area's own figures where those say so: such a block stays out of the area (56 products over K of 17 000 and more
// that went back to split-K by the current figures alone took 1.31 times as long with operands in cache, 1.43 from memory; 384 x
// 640 x 24064 NT 37 us and 52).  Else by the current ones, where they are far ahead: 120 sampled products 1.25 and 1.37 times as
// fast, the slowest 1.03 (512 x 768 x 31872 NN 111 us and 72).  Not from four ranges in TN, where the wave-K model is short by up to
// a half: ten products 0.71 to 0.98 times as fast (256 x 256 x 24576 48 us and 62), two 1.08 and 1.11.
static bool leaves_split_k(const Part& p, int64_t K, int layout, int64_t lda, int64_t ldb, double us, const WaveKChoice& wk) {
    if (wk.tile < 0) return false;
    if (wavek_choose(layout, p.m, p.n, K, lda, ldb, true).us < 0.97 * us) return true;
    return wk.us < 0.815 * us && !(layout == AXONN_TN && variants()[p.variant].splits >= 4);
}
// A block planned with split-K on the eight-wave kernel's tiles and counts instead.  700 sampled products that are planned so, on all of
// them (in cache, three sets in turn, from memory): 1.31, 1.31 and 1.53 times as fast as planned with 128 x 128 tiles (527, three of them 3-4 % slower),
// half tiles 1.12 to 1.17 where the models put it 2 % ahead, 256 x 256 tiles in four and more ranges 1.16 to 1.27; in two and three ranges 0.78 to
// 0.85, an output that has a round of large tiles nearly full.  Nor where NT would keep its 256 x 128 tiles in two ranges: the exchange saves least
// there and the ranges are long, over which the four-wave tile is 2 to 7 % ahead in all of the 12 sampled (256 x 14080 x 15488 132 us and 142), while three
// ranges gain 1.01 to 1.04.
static GroupSplitChoice split_on_eight_waves(const Part& p, int64_t K, int layout, double us) {
    const Variant& x = variants()[p.variant];
    const int area = x.bm * x.bn;
    if (us <= 0.0 || (area == 256 * 256 && x.splits < 4)) return GroupSplitChoice{};
    const GroupSplitChoice c = group_split_choose(layout, p.m, p.n, K, kStaticSlots * kSlotBytes, kMaxFlags);
    if (c.tile < 0 || c.us >= (area <= 128 * 128 ? 1.1 : 0.98) * us) return GroupSplitChoice{};
    int rows = 0, cols = 0;
    group_split_tile(c, &rows, &cols);
    return layout == AXONN_NT && area == 256 * 128 && rows * cols == area && x.splits == 2 && c.splits == 2 ? GroupSplitChoice{} : c;
}
static void settle_parts(Plan& plan, int64_t M, int64_t N, int64_t K, int layout) {
    const int64_t lda = layout == AXONN_TN ? M : K, ldb = layout == AXONN_NT ? K : N;
    for (int i = 0; i < plan.parts; ++i) {
        Part& p = plan.part[i];
        if (variants()[p.variant].edge) {
            p.how = guarded_choice(p.row0, p.col0, p.m, p.n, M, N, K, layout);
        } else if (p.variant > 0) {
            const WaveKChoice wk = wavek_choose(layout, p.m, p.n, K, lda, ldb);
            if (variants()[p.variant].splits > 1) {
                const double us = block_us(p.variant, p.m, p.n, K, layout, lda, ldb, N);   // the same by either figures
                if (us > 0.0 && leaves_split_k(p, K, layout, lda, ldb, us, wk)) p.how.wavek = wk;
                else p.how.split = split_on_eight_waves(p, K, layout, us);
                continue;
            }
            const double us = tiles_us(p, M, N, K, layout);
            if (us <= 0.0) continue;
            BlockChoice best;
            best.us = 0.98 * us;
            if (wk.tile >= 0 && wk.us < best.us) {
                best.wavek = wk;
                best.us = wk.us;
            }
            tiles_choice(p.m, p.n, K, layout, lda, ldb, N, best, true);
            if (best.tile != p.variant) p.how = best;
        }
    }
}

// Plans are remembered per shape: the search above costs a few hundred model evaluations.
static std::map<std::tuple<int64_t, int64_t, int64_t, int, bool>, Plan> g_plans;
static std::mutex g_plans_mutex;

static Plan cached_plan(int64_t M, int64_t N, int64_t K, int layout, bool allow_split) {
    const auto key = std::make_tuple(M, N, K, layout, allow_split);
    {
        std::lock_guard<std::mutex> lock(g_plans_mutex);
        const auto it = g_plans.find(key);
        if (it != g_plans.end()) return it->second;
    }
    Plan plan = make_plan(M, N, K, layout, allow_split);
    settle_parts(plan, M, N, K, layout);
    std::lock_guard<std::mutex> lock(g_plans_mutex);
    if (g_plans.size() >= 4096) g_plans.clear();
    g_plans[key] = plan;
    return plan;
}

static int check_args(int64_t M, int64_t N, int64_t K, int layout, const void* a, const void* b,
                      void* c, int fp32_accumulate) {
    constexpr int64_t kMaxDim = (int64_t)1 << 31, kMaxElems = (int64_t)1 << 40;
    if (M < 0 || N < 0 || K < 0 || M >= kMaxDim || N >= kMaxDim || K >= kMaxDim) return AXONN_ERR_INVALID_ARG;
    if (layout < 0 || layout > 2) return AXONN_ERR_INVALID_ARG;
    if (fp32_accumulate != 0 && fp32_accumulate != 1) return AXONN_ERR_INVALID_ARG;
    if (M * K >= kMaxElems || K * N >= kMaxElems || M * N >= kMaxElems) return AXONN_ERR_INVALID_ARG;
    if (M == 0 || N == 0) return AXONN_OK;
    if (!c || (reinterpret_cast<uintptr_t>(c) & 15)) return AXONN_ERR_INVALID_ARG;
    if (K > 0) {
        if (!a || !b) return AXONN_ERR_INVALID_ARG;
        if ((reinterpret_cast<uintptr_t>(a) & 15) || (reinterpret_cast<uintptr_t>(b) & 15))
            return AXONN_ERR_INVALID_ARG;
    }
    return AXONN_OK;
}

static void raise_lds_limits() {
    for (const Variant& var : variants())
        for (int l = 0; l < 3; ++l)
            for (const tile_kernel_t fn : {var.fn[l], var.fn_tail[l]})
                if (fn) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, var.lds_bytes);
    edge_kernel_raise_lds_limit();
    wavek_raise_lds_limit();
    group_raise_lds_limit();
    (void)hipGetLastError();
}

// once per device, the first time a kernel that needs it is about to be launched there
static void raise_lds_limits_once() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        raise_lds_limits();
        return;
    }
    std::call_once(g_attr_once[dev], raise_lds_limits);
}

// What the launches touch of it: nothing for a block planned with split-K that runs on a kernel without it.
static size_t split_bytes_run(const Plan& plan) {
    size_t bytes = 0;
    for (int i = 0; i < plan.parts; ++i)
        if (plan.part[i].how.wavek.tile < 0 && plan.part[i].how.group.tile < 0 && plan.part[i].how.tile < 0) bytes = std::max(bytes, split_bytes(plan.part[i]));
    return bytes;
}

// workgroups of the launch over block `p`
static int64_t part_workgroups(const Part& p) {
    const Variant& var = variants()[p.variant];
    return ((p.m + var.bm - 1) / var.bm) * ((p.n + var.bn - 1) / var.bn) * var.splits;
}

static uint32_t next_epoch() {
    for (;;) {
        const uint32_t epoch = g_epoch.fetch_add(1, std::memory_order_relaxed) + 1;
        if (epoch != 0 && epoch != ~0u) return epoch;   // flags start at 0; ~epoch: see split_exchange.hpp
    }
}

// A tile kernel over the m x n block that starts at A, B, C.
static void launch_tiles(const Variant& var, int64_t m, int64_t n, int64_t K, int layout, const uint16_t* A, const uint16_t* B,
                         uint16_t* C, int64_t lda, int64_t ldb, int64_t ldc, const Scratch& scratch, hipStream_t s) {
    const int tiles_m = (int)((m + var.bm - 1) / var.bm), tiles_n = (int)((n + var.bn - 1) / var.bn);
    const int64_t tiles = (int64_t)tiles_m * tiles_n;
    const int group_m = tiles_m < 8 ? tiles_m : 8;
    SplitK sk{nullptr, nullptr, nullptr, 0u, 1, 0};
    if (var.splits > 1) {
        const uint32_t epoch = next_epoch();
        // one iteration less for every writer (measured on 2048 x 4096 x 4096 and x 16384 in two ranges: 64 k
        // takes 1-2 us off, 128 and more give it back)
        const int skew = (var.k64 && K / var.splits >= 1024) ? TileCfgK64::KS : 0;
        sk = SplitK{scratch.partials, scratch.flags, scratch.timeouts(), epoch, var.splits, skew};
    }
    const int64_t grid = var.resident > 0 ? std::min<int64_t>(tiles, var.resident) : tiles * var.splits;
    const int k_tail = (int)(K % 64);
    hipLaunchKernelGGL(k_tail ? var.fn_tail[layout] : var.fn[layout], dim3((unsigned)grid), dim3(var.threads), var.lds_bytes, s,
                       A, B, C, (int)(K - k_tail + (k_tail ? 64 : 0)), (int)lda, (int)ldb, (int)ldc,
                       TileGrid{tiles_m, tiles_n, (int)(m - var.bm), (int)(n - var.bn), k_tail}, group_m, sk);
}

// One kernel launch over the block `p` of the M x N output.
static void launch_part(const Part& p, int64_t M, int64_t N, int64_t K, int layout, const uint16_t* A, const uint16_t* B,
                        uint16_t* C, const Scratch& scratch, uint32_t probes, hipStream_t s) {
    const Variant& var = variants()[p.variant];
    const int64_t lda = layout == AXONN_TN ? M : K, ldb = layout == AXONN_NT ? K : N, ldc = N;
    A += layout == AXONN_TN ? p.row0 : p.row0 * K;
    B += layout == AXONN_NT ? p.col0 * K : p.col0;
    C += p.row0 * N + p.col0;
    if (p.how.wavek.tile >= 0) {
        const int64_t dm = p.how.lead_m, dn = p.how.lead_n;
        wavek_launch(p.how.wavek, layout, s, A - (layout == AXONN_TN ? dm : dm * K), B - (layout == AXONN_NT ? dn * K : dn),
                     C - dm * N - dn, p.m + dm, p.n + dn, K, lda, ldb, ldc);
        return;
    }
    if (p.how.group.tile >= 0) {
        group_launch(p.how.group, layout, s, A, B, C, p.m, p.n, K, lda, ldb, ldc);
        return;
    }
    if (p.how.split.tile >= 0) {
        group_split_launch(p.how.split, layout, s, A, B, C, p.m, p.n, K, lda, ldb, ldc, scratch.partials, scratch.flags, next_epoch(), probes);
        return;
    }
    if (var.edge && p.how.tile < 0) {
        const int tiles_n = (int)((p.n + var.bn - 1) / var.bn);
        edge_kernel_launch(layout, (unsigned)part_workgroups(p), s, A, B, C, p.m, p.n, K, lda, ldb, ldc, tiles_n);
        return;
    }
    launch_tiles(p.how.tile >= 0 ? variants()[p.how.tile] : var, p.m, p.n, K, layout, A, B, C, lda, ldb, ldc, scratch, s);
}

// Where a call's split-K kernels find their scratch area.
enum class ScratchFrom { Registered, Static };

// The launches of a call made now on the current device, and the scratch area that its split-K kernels use.
static int plan_call(int64_t M, int64_t N, int64_t K, int layout, ScratchFrom from, Plan& plan, Scratch& scratch) {
    const int forced = g_forced.load(std::memory_order_relaxed);
    if (forced >= 0) {
        if (!variant_supports(forced, M, N, K, layout)) return AXONN_ERR_UNSUPPORTED;
        plan = Plan{1, {{forced, M, N, 0, 0}}};   // that very kernel (for the last variant: gemm_edge_kernel)
    } else {
        plan = cached_plan(M, N, K, layout, g_split_k_enabled.load(std::memory_order_relaxed) != 0);
    }
    if (const size_t need = split_bytes_run(plan)) {
        if (from == ScratchFrom::Static) {
            // the static area has one size: a product whose plan needs more is refused, not re-planned
            if (need > kStaticSlots * kSlotBytes || !(scratch = static_scratch()).partials) return AXONN_ERR_WORKSPACE;
        } else if (!(scratch = registered_scratch(need)).partials) {
            if (forced >= 0) return AXONN_ERR_WORKSPACE;
            plan = cached_plan(M, N, K, layout, false);   // no area, or too small a one: the kernels that need none
        }
        // the eight-wave kernel's partial sums may take more than the variant's: where the area is short of them, the variant itself
        for (int i = 0; i < plan.parts; ++i)
            if (group_split_bytes(plan.part[i].how.split, plan.part[i].m, plan.part[i].n) > scratch.partial_bytes) plan.part[i].how.split = GroupSplitChoice{};
    }
    return AXONN_OK;
}

// The kernel behind one launch, named as profile_summary.short() names its symbol (plus the number of K ranges
// or of waves per tile, which are run-time arguments).  A plan names variants: what runs is more than that.
static int part_kernel_name(const Part& p, int64_t N, int64_t K, int layout, char* name, size_t bytes) {
    const Variant& planned = variants()[p.variant];
    if (p.how.wavek.tile >= 0) {
        int rows = 0, cols = 0;
        wavek_tile(p.how.wavek, &rows, &cols);
        const ShortK short_k = wavek_short(p.how.wavek, layout, p.m + p.how.lead_m, p.n + p.how.lead_n, K, N);
        if (short_k != ShortK::No)
            return std::snprintf(name, bytes, "wavek_%dx%d_k%d%s", rows, cols, K <= 32 ? 32 : 64, short_k == ShortK::Chunks ? "_xcd" : "");
        return std::snprintf(name, bytes, "wavek_%dx%d_w%d", rows, cols, p.how.wavek.waves);
    }
    const char* const tail = planned.bm && K % 64 ? "_ktail" : "";
    if (p.how.group.tile >= 0) {
        int rows = 0, cols = 0, groups = 0;
        group_tile(p.how.group, &rows, &cols, &groups);
        return std::snprintf(name, bytes, "mfma16k64g_%dx%d%s%s", rows, cols, groups == 2 ? "_g2" : "", tail);
    }
    if (p.how.split.tile >= 0) {
        int rows = 0, cols = 0;
        group_split_tile(p.how.split, &rows, &cols);
        return std::snprintf(name, bytes, "mfma16k64g_%dx%d_sk%d", rows, cols, p.how.split.splits);
    }
    if (planned.edge && p.how.tile < 0) return std::snprintf(name, bytes, "edge_%dx%d", planned.bm, planned.bn);
    const Variant& var = p.how.tile >= 0 ? variants()[p.how.tile] : planned;
    if (var.group) return std::snprintf(name, bytes, "mfma16k64g_%dx%d%s", var.bm, var.bn, tail);   // one kernel behind the variants of a tile
    // 128 x 128 tiles of two K-contiguous operands (NT) with split-K: the 64-k kernel
    const bool k64_under_ring_name = layout == AXONN_NT && !var.k64 && var.bm == 128 && var.bn == 128;
    return std::snprintf(name, bytes, "%s%s%s", k64_under_ring_name ? "mfma16k64_" : "",
                         var.name + (k64_under_ring_name ? std::strlen("mfma16_") : 0), tail);
}

static int launch(int64_t M, int64_t N, int64_t K, int layout, const void* a, const void* b, void* c,
                  int fp32_accumulate, void* stream, ScratchFrom from = ScratchFrom::Registered, uint32_t probes = kGroupSplitProbes) {
    const int rc = check_args(M, N, K, layout, a, b, c, fp32_accumulate);
    if (rc != AXONN_OK) return rc;
    if (M == 0 || N == 0) return AXONN_OK;

    Plan plan;
    Scratch scratch;
    const int planned = plan_call(M, N, K, layout, from, plan, scratch);
    if (planned != AXONN_OK) return planned;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint16_t* A = static_cast<const uint16_t*>(a);
    const uint16_t* B = static_cast<const uint16_t*>(b);
    uint16_t* C = static_cast<uint16_t*>(c);

    (void)hipGetLastError();
    if (variants()[plan.part[0].variant].bm == 0) {
        const int64_t blocks = ((M + 15) / 16) * ((N + 15) / 16);
        const dim3 grid((unsigned)std::min<int64_t>(blocks, (int64_t)1 << 20));
        switch (layout) {
            case AXONN_NN: hipLaunchKernelGGL(gemm_naive_kernel<AXONN_NN>, grid, dim3(256), 0, s, A, B, C, M, N, K); break;
            case AXONN_NT: hipLaunchKernelGGL(gemm_naive_kernel<AXONN_NT>, grid, dim3(256), 0, s, A, B, C, M, N, K); break;
            default:       hipLaunchKernelGGL(gemm_naive_kernel<AXONN_TN>, grid, dim3(256), 0, s, A, B, C, M, N, K); break;
        }
    } else {
        raise_lds_limits_once();
        for (int i = 0; i < plan.parts; ++i)
            if (part_workgroups(plan.part[i]) >= ((int64_t)1 << 31)) return AXONN_ERR_UNSUPPORTED;
        for (int i = 0; i < plan.parts; ++i) launch_part(plan.part[i], M, N, K, layout, A, B, C, scratch, probes, s);
    }
    return hipGetLastError() == hipSuccess ? AXONN_OK : AXONN_ERR_LAUNCH;
}

// ------------------------------------------------------------------------------------------
// Mode tuner (paper Sec. IV-C): time a product in all three modes once, remember the result.
// ------------------------------------------------------------------------------------------
static std::map<std::tuple<int, int64_t, int64_t, int64_t>, axonn_tune_result_t> g_tuned;
static std::mutex g_tuned_mutex;

static bool first_is_mk(int mode) { return mode != AXONN_TN; }
static bool second_is_kn(int mode) { return mode != AXONN_NT; }

// Mean time in microseconds of `reps` runs of f() on stream s (after `warm` untimed ones); < 0 on error.
template <class F>
static float time_us(hipStream_t s, int warm, int reps, F&& f) {
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return -1.f;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return -1.f;
    }
    bool ok = true;
    for (int i = 0; i < warm && ok; ++i) ok = f() == AXONN_OK;
    ok = ok && hipEventRecord(e0, s) == hipSuccess;
    for (int i = 0; i < reps && ok; ++i) ok = f() == AXONN_OK;
    ok = ok && hipEventRecord(e1, s) == hipSuccess && hipEventSynchronize(e1) == hipSuccess;
    float ms = 0.f;
    ok = ok && hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return ok ? ms * 1000.f / (float)reps : -1.f;
}

}  // namespace axonn

extern "C" {

int axonn_linear_tune(int op, int64_t M, int64_t N, int64_t K, const void* first, const void* second, void* out,
                      void* scratch, size_t scratch_bytes, void* stream, axonn_tune_result_t* result) {
    using namespace axonn;
    if (op < 0 || op > 2 || !result || M <= 0 || N <= 0 || K <= 0) return AXONN_ERR_INVALID_ARG;
    const int nat = op;   // fwd: NN, bwd_data: NT, bwd_weight: TN -- the modes the cached buffers give for free
    int rc = check_args(M, N, K, nat, first, second, out, 1);
    if (rc != AXONN_OK) return rc;
    if (scratch_bytes && (!scratch || (reinterpret_cast<uintptr_t>(scratch) & 255))) return AXONN_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t first_bytes = (((size_t)M * K * 2) + 255) & ~(size_t)255, second_bytes = (size_t)K * N * 2;
    axonn_tune_result_t r;
    r.best_layout = r.best_layout_all_in = nat;
    float best = -1.f, best_all = -1.f;
    for (int m = 0; m < 3; ++m) {
        r.gemm_us[m] = -1.f;
        r.restore_first_us[m] = r.restore_second_us[m] = 0.f;
        const bool tf = first_is_mk(m) != first_is_mk(nat), ts = second_is_kn(m) != second_is_kn(nat);
        const size_t need = (tf ? first_bytes : 0) + (ts ? second_bytes : 0);
        if (need > scratch_bytes) continue;   // this mode cannot be tried
        const void* a = first;
        const void* b = second;
        char* free_ptr = static_cast<char*>(scratch);
        if (tf) {
            const int64_t rows = first_is_mk(nat) ? M : K, cols = first_is_mk(nat) ? K : M;
            void* dst = free_ptr;
            free_ptr += first_bytes;
            r.restore_first_us[m] = time_us(s, 1, 3, [&] { return axonn_transpose_bf16(rows, cols, first, dst, stream); });
            if (r.restore_first_us[m] < 0.f) return AXONN_ERR_LAUNCH;
            a = dst;
        }
        if (ts) {
            const int64_t rows = second_is_kn(nat) ? K : N, cols = second_is_kn(nat) ? N : K;
            void* dst = free_ptr;
            r.restore_second_us[m] = time_us(s, 1, 3, [&] { return axonn_transpose_bf16(rows, cols, second, dst, stream); });
            if (r.restore_second_us[m] < 0.f) return AXONN_ERR_LAUNCH;
            b = dst;
        }
        r.gemm_us[m] = time_us(s, 2, 5, [&] { return launch(M, N, K, m, a, b, out, 1, stream); });
        if (r.gemm_us[m] < 0.f) return AXONN_ERR_LAUNCH;
        // the weight (second operand of fwd and bwd_data) changes once per optimiser step, the other
        // operands with every call: only their re-storage is charged to the call
        const float all_in = r.gemm_us[m] + r.restore_first_us[m] + (op == 2 ? r.restore_second_us[m] : 0.f);
        if (best < 0.f || r.gemm_us[m] < best) {
            best = r.gemm_us[m];
            r.best_layout = m;
        }
        if (best_all < 0.f || all_in < best_all) {
            best_all = all_in;
            r.best_layout_all_in = m;
        }
    }
    {
        std::lock_guard<std::mutex> lock(g_tuned_mutex);
        g_tuned[std::make_tuple(op, M, N, K)] = r;
    }
    *result = r;
    return AXONN_OK;
}

int axonn_linear_tuned(int op, int64_t M, int64_t N, int64_t K, axonn_tune_result_t* result) {
    if (op < 0 || op > 2 || !result) return AXONN_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(axonn::g_tuned_mutex);
    auto it = axonn::g_tuned.find(std::make_tuple(op, M, N, K));
    if (it == axonn::g_tuned.end()) return 0;
    *result = it->second;
    return 1;
}

int axonn_linear_tuned_set(int op, int64_t M, int64_t N, int64_t K, const axonn_tune_result_t* result) {
    if (op < 0 || op > 2 || !result || M <= 0 || N <= 0 || K <= 0 || result->best_layout < 0 || result->best_layout > 2 ||
        result->best_layout_all_in < 0 || result->best_layout_all_in > 2)
        return AXONN_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(axonn::g_tuned_mutex);
    axonn::g_tuned[std::make_tuple(op, M, N, K)] = *result;
    return AXONN_OK;
}

int axonn_linear_tuned_call(int op, int64_t M, int64_t N, int64_t K, const void* first, const void* second, void* out,
                            const void* second_restored, void* scratch, size_t scratch_bytes, int fp32_accumulate,
                            void* stream, int* layout_used) {
    using namespace axonn;
    if (op < 0 || op > 2) return AXONN_ERR_INVALID_ARG;
    const int nat = op;
    int rc = check_args(M, N, K, nat, first, second, out, fp32_accumulate);
    if (rc != AXONN_OK) return rc;
    if (scratch_bytes && (!scratch || (reinterpret_cast<uintptr_t>(scratch) & 255))) return AXONN_ERR_INVALID_ARG;
    if (second_restored && (reinterpret_cast<uintptr_t>(second_restored) & 15)) return AXONN_ERR_INVALID_ARG;
    int mode = nat;
    {
        std::lock_guard<std::mutex> lock(g_tuned_mutex);
        const auto it = g_tuned.find(std::make_tuple(op, M, N, K));
        if (it != g_tuned.end()) mode = it->second.best_layout_all_in;
    }
    bool tf = first_is_mk(mode) != first_is_mk(nat), ts = second_is_kn(mode) != second_is_kn(nat);
    const size_t first_bytes = (((size_t)M * K * 2) + 255) & ~(size_t)255, second_bytes = (size_t)K * N * 2;
    const size_t need = (tf ? first_bytes : 0) + ((ts && !second_restored) ? second_bytes : 0);
    if (need > scratch_bytes || M == 0 || N == 0 || K == 0) {   // no room to re-store: the natural mode needs none
        mode = nat;
        tf = ts = false;
    }
    const void* a = first;
    const void* b = second;
    char* free_ptr = static_cast<char*>(scratch);
    if (tf) {
        const int64_t rows = first_is_mk(nat) ? M : K, cols = first_is_mk(nat) ? K : M;
        rc = axonn_transpose_bf16(rows, cols, first, free_ptr, stream);
        if (rc != AXONN_OK) return rc;
        a = free_ptr;
        free_ptr += first_bytes;
    }
    if (ts) {
        if (second_restored) {
            b = second_restored;
        } else {
            const int64_t rows = second_is_kn(nat) ? K : N, cols = second_is_kn(nat) ? N : K;
            rc = axonn_transpose_bf16(rows, cols, second, free_ptr, stream);
            if (rc != AXONN_OK) return rc;
            b = free_ptr;
        }
    }
    if (layout_used) *layout_used = mode;
    return launch(M, N, K, mode, a, b, out, fp32_accumulate, stream);
}

void axonn_linear_tune_reset(void) {
    std::lock_guard<std::mutex> lock(axonn::g_tuned_mutex);
    axonn::g_tuned.clear();
}

int axonn_linear_fwd(int64_t M, int64_t N, int64_t K, int layout, const void* X, const void* W, void* Y,
                     int fp32_accumulate, void* stream) {
    return axonn::launch(M, N, K, layout, X, W, Y, fp32_accumulate, stream);
}

int axonn_linear_bwd_data(int64_t M, int64_t N, int64_t K, int layout, const void* dY, const void* W, void* dX,
                          int fp32_accumulate, void* stream) {
    return axonn::launch(M, N, K, layout, dY, W, dX, fp32_accumulate, stream);
}

int axonn_linear_bwd_weight(int64_t M, int64_t N, int64_t K, int layout, const void* X, const void* dY, void* dW,
                            int fp32_accumulate, void* stream) {
    return axonn::launch(M, N, K, layout, X, dY, dW, fp32_accumulate, stream);
}

int axonn_linear_gemm_static(int64_t M, int64_t N, int64_t K, int layout, const void* first, const void* second, void* out,
                             int fp32_accumulate, void* stream) {
    return axonn::launch(M, N, K, layout, first, second, out, fp32_accumulate, stream, axonn::ScratchFrom::Static);
}

int axonn_linear_gemm_split_probes(int64_t M, int64_t N, int64_t K, int layout, const void* first, const void* second, void* out,
                                   uint32_t probes, void* stream) {
    const int rc = axonn::check_args(M, N, K, layout, first, second, out, 1);
    if (rc != AXONN_OK) return rc;
    if (M == 0 || N == 0) return AXONN_ERR_UNSUPPORTED;
    axonn::Plan plan;
    axonn::Scratch scratch;
    const int planned = axonn::plan_call(M, N, K, layout, axonn::ScratchFrom::Registered, plan, scratch);
    if (planned != AXONN_OK) return planned;
    for (int i = 0; i < plan.parts; ++i)
        if (plan.part[i].how.split.tile >= 0) return axonn::launch(M, N, K, layout, first, second, out, 1, stream, axonn::ScratchFrom::Registered, probes);
    return AXONN_ERR_UNSUPPORTED;
}

size_t axonn_linear_static_scratch_bytes(void) { return axonn::kStaticBytes; }

const char* axonn_status_string(int status) {
    switch (status) {
        case AXONN_OK: return "ok";
        case AXONN_ERR_INVALID_ARG: return "invalid argument (null or misaligned pointer, bad dimension, layout or flag)";
        case AXONN_ERR_UNSUPPORTED: return "the forced kernel variant cannot run this shape";
        case AXONN_ERR_LAUNCH: return "the HIP runtime refused the kernel launch";
        case AXONN_ERR_WORKSPACE: return "no split-K scratch area of the size needed (none registered, the registered one too small, or the product's plan exceeds the static area)";
        default: return "unknown status";
    }
}

int axonn_linear_version(void) { return 100; }

int axonn_linear_num_variants(void) { return axonn::num_variants(); }

const char* axonn_linear_variant_name(int variant) {
    return (variant >= 0 && variant < axonn::num_variants()) ? axonn::variants()[variant].name : nullptr;
}

int axonn_linear_variant_supports(int variant, int64_t M, int64_t N, int64_t K, int layout) {
    return axonn::variant_supports(variant, M, N, K, layout) ? 1 : 0;
}

int axonn_linear_select_variant(int64_t M, int64_t N, int64_t K, int layout) {
    if (M < 0 || N < 0 || K < 0 || layout < 0 || layout > 2) return AXONN_ERR_INVALID_ARG;
    return axonn::select_variant(M, N, K, layout, axonn::g_split_k_enabled.load(std::memory_order_relaxed) != 0);
}

int axonn_linear_plan(int64_t M, int64_t N, int64_t K, int layout, axonn_plan_part_t parts[AXONN_MAX_PLAN_PARTS]) {
    if (M <= 0 || N <= 0 || K < 0 || layout < 0 || layout > 2 || !parts) return AXONN_ERR_INVALID_ARG;
    const axonn::Plan plan = axonn::cached_plan(M, N, K, layout, axonn::g_split_k_enabled.load(std::memory_order_relaxed) != 0);
    for (int i = 0; i < plan.parts; ++i)
        parts[i] = axonn_plan_part_t{plan.part[i].variant, plan.part[i].m, plan.part[i].n, plan.part[i].row0, plan.part[i].col0};
    return plan.parts;
}

int axonn_linear_call_plan(int64_t M, int64_t N, int64_t K, int layout, axonn_plan_part_t parts[AXONN_MAX_PLAN_PARTS]) {
    if (M <= 0 || N <= 0 || K < 0 || layout < 0 || layout > 2 || !parts) return AXONN_ERR_INVALID_ARG;
    axonn::Plan plan = axonn::cached_plan(M, N, K, layout, axonn::g_split_k_enabled.load(std::memory_order_relaxed) != 0);
    if (const size_t need = axonn::split_bytes_run(plan))
        if (!axonn::registered_scratch(need).partials) plan = axonn::cached_plan(M, N, K, layout, false);
    for (int i = 0; i < plan.parts; ++i)
        parts[i] = axonn_plan_part_t{plan.part[i].variant, plan.part[i].m, plan.part[i].n, plan.part[i].row0, plan.part[i].col0};
    return plan.parts;
}

int axonn_linear_part_kernel(int64_t M, int64_t N, int64_t K, int layout, int now, int part, char* name, size_t name_bytes) {
    if (M <= 0 || N <= 0 || K < 0 || layout < 0 || layout > 2 || (now != 0 && now != 1) || part < 0 || !name || name_bytes == 0)
        return AXONN_ERR_INVALID_ARG;
    axonn::Plan plan;
    if (now) {
        axonn::Scratch scratch;
        const int rc = axonn::plan_call(M, N, K, layout, axonn::ScratchFrom::Registered, plan, scratch);
        if (rc != AXONN_OK) return rc;
    } else {
        plan = axonn::cached_plan(M, N, K, layout, axonn::g_split_k_enabled.load(std::memory_order_relaxed) != 0);
        // with the scratch area that axonn_linear_workspace_bytes asks for: the variants' own kernels
        for (int i = 0; i < plan.parts; ++i) plan.part[i].how.split = axonn::GroupSplitChoice{};
    }
    if (part >= plan.parts) return AXONN_ERR_INVALID_ARG;
    const int n = axonn::part_kernel_name(plan.part[part], N, K, layout, name, name_bytes);
    return n > 0 && (size_t)n < name_bytes ? plan.parts : AXONN_ERR_INVALID_ARG;
}

int axonn_linear_init(void) {
    axonn::raise_lds_limits_once();
    return axonn::static_scratch().partials ? AXONN_OK : AXONN_ERR_WORKSPACE;
}

size_t axonn_linear_workspace_bytes(int64_t M, int64_t N, int64_t K, int layout) {
    if (M <= 0 || N <= 0 || K <= 0 || layout < 0 || layout > 2) return 0;
    const size_t bytes = axonn::split_bytes(axonn::cached_plan(M, N, K, layout, true));
    // never less than what axonn_linear_set_workspace accepts (a plan of 128 x 128 tiles can need less)
    return bytes ? axonn::kFlagBytes + std::max(bytes, axonn::kSlotBytes) : 0;
}

int axonn_linear_set_workspace(void* dev_ptr, size_t bytes) {
    if ((dev_ptr == nullptr) != (bytes == 0) || (reinterpret_cast<uintptr_t>(dev_ptr) & 255)) return AXONN_ERR_INVALID_ARG;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= axonn::kMaxDevices) return AXONN_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(axonn::g_scratch_mutex);
    axonn::Scratch& sc = axonn::g_scratch[dev];
    if (dev_ptr == nullptr) {            // unregistered: from now on the kernels that need no scratch
        sc = axonn::Scratch{};
        return AXONN_OK;
    }
    if (bytes < axonn::kFlagBytes + axonn::kSlotBytes) return AXONN_ERR_WORKSPACE;
    // flags start at zero (a flag is valid when it equals the launch's non-zero epoch)
    if (hipMemset(dev_ptr, 0, axonn::kFlagBytes) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
        (void)hipGetLastError();
        return AXONN_ERR_WORKSPACE;
    }
    sc = axonn::carve(dev_ptr, bytes);
    return AXONN_OK;
}

int axonn_linear_set_split_k(int enable) {
    if (enable != 0 && enable != 1) return AXONN_ERR_INVALID_ARG;
    return axonn::g_split_k_enabled.exchange(enable, std::memory_order_relaxed);
}

int axonn_linear_split_k_timeouts(uint64_t* count) {
    if (!count) return AXONN_ERR_INVALID_ARG;
    *count = 0;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= axonn::kMaxDevices) return AXONN_ERR_LAUNCH;
    uint32_t* counters[2] = {nullptr, nullptr};   // the registered area's and the static area's
    {
        std::lock_guard<std::mutex> lock(axonn::g_scratch_mutex);
        if (axonn::g_scratch[dev].flags) counters[0] = axonn::g_scratch[dev].timeouts();
    }
    {
        std::lock_guard<std::mutex> lock(axonn::g_static_mutex);
        if (axonn::g_static_ptr[dev]) counters[1] = axonn::carve(axonn::g_static_ptr[dev], axonn::kStaticBytes).timeouts();
    }
    for (uint32_t* counter : counters) {
        if (!counter) continue;   // no split-K kernel has used that area on this device
        uint32_t v = 0;
        if (hipMemcpy(&v, counter, sizeof v, hipMemcpyDeviceToHost) != hipSuccess) {
            (void)hipGetLastError();
            return AXONN_ERR_LAUNCH;
        }
        *count += v;
    }
    return AXONN_OK;
}

int axonn_transpose_bf16(int64_t rows, int64_t cols, const void* src, void* dst, void* stream) {
    constexpr int64_t kMaxDim = (int64_t)1 << 31, kMaxElems = (int64_t)1 << 40;
    if (rows < 0 || cols < 0 || rows >= kMaxDim || cols >= kMaxDim || rows * cols >= kMaxElems) return AXONN_ERR_INVALID_ARG;
    if (rows == 0 || cols == 0) return AXONN_OK;
    const uintptr_t s = reinterpret_cast<uintptr_t>(src), d = reinterpret_cast<uintptr_t>(dst);
    const uintptr_t bytes = (uintptr_t)rows * (uintptr_t)cols * 2;
    if (!src || !dst || (s & 1) || (d & 1) || (s < d + bytes && d < s + bytes)) return AXONN_ERR_INVALID_ARG;
    const axonn::TrKernel kernel = axonn::tr_choose(rows, cols, s, d);
    if (kernel == axonn::TrKernel::Refused) return AXONN_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint16_t* from = static_cast<const uint16_t*>(src);
    uint16_t* to = static_cast<uint16_t*>(dst);
    (void)hipGetLastError();
    if (kernel == axonn::TrKernel::Element) {
        hipLaunchKernelGGL(axonn::transpose_naive_kernel, dim3((unsigned)((rows + 63) / 64), (unsigned)((cols + 3) / 4)), dim3(256), 0, st,
                           from, to, rows, cols);
    } else if (kernel == axonn::TrKernel::Window) {
        const int64_t tiles_r = axonn::tr_windows(rows), tiles_c = axonn::tr_tiles(cols);
        hipLaunchKernelGGL(axonn::transpose_window_kernel, dim3((unsigned)(tiles_r * tiles_c)), dim3(axonn::TR_WINDOW_THREADS), 0, st,
                           from, to, rows, cols, (int)tiles_r, (int)tiles_c);
    } else {
        const int64_t tiles_r = axonn::tr_tiles(rows), tiles_c = axonn::tr_tiles(cols);   // product below 2^29: rows * cols < 2^40
        hipLaunchKernelGGL(kernel == axonn::TrKernel::TileBands ? axonn::transpose_tile_kernel<true> : axonn::transpose_tile_kernel<false>,
                           dim3((unsigned)(tiles_r * tiles_c)), dim3(256), 0, st, from, to, rows, cols, (int)tiles_r, (int)tiles_c);
    }
    return hipGetLastError() == hipSuccess ? AXONN_OK : AXONN_ERR_LAUNCH;
}

const char* axonn_transpose_kernel_at(int64_t rows, int64_t cols, const void* src, const void* dst) {
    if (rows <= 0 || cols <= 0) return nullptr;
    switch (axonn::tr_choose(rows, cols, reinterpret_cast<uintptr_t>(src), reinterpret_cast<uintptr_t>(dst))) {
        case axonn::TrKernel::Element: return "transpose_naive";
        case axonn::TrKernel::Tile: return "transpose_tile";
        case axonn::TrKernel::TileBands: return "transpose_tile_bands";
        case axonn::TrKernel::Window: return "transpose_window";
        default: return nullptr;
    }
}

const char* axonn_transpose_kernel(int64_t rows, int64_t cols, int aligned) {
    const void* const at = reinterpret_cast<const void*>(static_cast<uintptr_t>(aligned ? 128 : 130));
    return axonn_transpose_kernel_at(rows, cols, at, at);
}

static bool comm_args_ok(const int* grid, int g_node, double beta_inter, double bytes_per_element) {
    if (!grid || g_node < 1 || !(beta_inter > 0.0) || !(bytes_per_element > 0.0)) return false;
    for (int i = 0; i < 4; ++i)
        if (grid[i] < 1) return false;
    return true;
}

int axonn_comm_group_bandwidths(const int* grid, int g_node, double beta_inter, const double* intra_bw, double* beta_out) {
    if (!comm_args_ok(grid, g_node, beta_inter, 1.0) || !beta_out) return AXONN_ERR_INVALID_ARG;
    return axonn::comm_group_bandwidths(grid, g_node, beta_inter, intra_bw, beta_out) ? AXONN_OK : AXONN_ERR_INVALID_ARG;
}

int axonn_comm_layer_time(const axonn_comm_layer_t* layer, const int* grid, const double* beta, double bytes_per_element,
                          double* terms_out) {
    if (!layer || !beta || !terms_out || !comm_args_ok(grid, 1, 1.0, bytes_per_element)) return AXONN_ERR_INVALID_ARG;
    if (layer->m < 0 || layer->k < 0 || layer->n < 0) return AXONN_ERR_INVALID_ARG;
    for (int i = 0; i < 4; ++i)
        if (grid[i] > 1 && !(beta[i] > 0.0)) return AXONN_ERR_INVALID_ARG;
    axonn::comm_layer_terms(*layer, grid, beta, bytes_per_element, terms_out);
    return AXONN_OK;
}

int64_t axonn_comm_rank_grids(int64_t g_total, const axonn_comm_layer_t* layers, int n_layers, int g_node,
                              double beta_inter, const double* intra_bw, double bytes_per_element,
                              axonn_comm_grid_t* out, int64_t max_out) {
    const int one[4] = {1, 1, 1, 1};
    if (g_total < 1 || g_total > ((int64_t)1 << 30) || n_layers < 0 || (n_layers > 0 && !layers) || max_out < 0 ||
        (max_out > 0 && !out) || !comm_args_ok(one, g_node, beta_inter, bytes_per_element))
        return AXONN_ERR_INVALID_ARG;
    for (int l = 0; l < n_layers; ++l)
        if (layers[l].m < 0 || layers[l].k < 0 || layers[l].n < 0) return AXONN_ERR_INVALID_ARG;
    std::vector<int64_t> divs;
    for (int64_t d = 1; d * d <= g_total; ++d)
        if (g_total % d == 0) {
            divs.push_back(d);
            if (d != g_total / d) divs.push_back(g_total / d);
        }
    std::sort(divs.begin(), divs.end());
    std::vector<axonn_comm_grid_t> rows;
    for (int64_t gx : divs)
        for (int64_t gy : divs) {
            if ((g_total / gx) % gy) continue;
            const int64_t r2 = g_total / gx / gy;
            for (int64_t gz : divs) {
                if (r2 % gz) continue;
                const int grid[4] = {(int)gx, (int)gy, (int)gz, (int)(r2 / gz)};
                double beta[4], terms[6], total = 0.0;
                if (!axonn::comm_group_bandwidths(grid, g_node, beta_inter, intra_bw, beta)) return AXONN_ERR_INVALID_ARG;
                for (int l = 0; l < n_layers; ++l) {
                    axonn::comm_layer_terms(layers[l], grid, beta, bytes_per_element, terms);
                    total += terms[5];
                }
                rows.push_back(axonn_comm_grid_t{grid[0], grid[1], grid[2], grid[3], total});
            }
        }
    std::sort(rows.begin(), rows.end(), [](const axonn_comm_grid_t& a, const axonn_comm_grid_t& b) {
        if (a.seconds != b.seconds) return a.seconds < b.seconds;
        if (a.gx != b.gx) return a.gx < b.gx;
        if (a.gy != b.gy) return a.gy < b.gy;
        if (a.gz != b.gz) return a.gz < b.gz;
        return a.gdata < b.gdata;
    });
    const int64_t n_out = std::min<int64_t>(max_out, (int64_t)rows.size());
    for (int64_t i = 0; i < n_out; ++i) out[i] = rows[i];
    return (int64_t)rows.size();
}

int axonn_linear_force_variant(int variant) {
    if (variant < -1 || variant >= axonn::num_variants()) return AXONN_ERR_INVALID_ARG;
    axonn::g_forced.store(variant, std::memory_order_relaxed);
    return AXONN_OK;
}

}  // extern "C"
