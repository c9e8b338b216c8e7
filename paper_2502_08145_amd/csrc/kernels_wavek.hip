// Translation unit of the wave-K kernel (see kernels.hpp).
#include "kernels.hpp"
#include "gemm_wavek.hpp"

#include <cmath>

namespace axonn {

typedef void (*wavek_kernel_t)(const uint16_t*, const uint16_t*, uint16_t*, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int, int, int);

// The tiles that are built, in 16 x 16 blocks, per layout (NN, NT, TN).  An MN-contiguous operand wants at
// least two blocks side by side (a k-row of one block is 32 bytes of a 128-byte line); the 1 x 1 tile serves
// it only where the matrix is narrower than that.  Among 22 000 sampled products (outputs of 1 to 16384 rows, up to
// 30 GFLOP) the best of these tiles is within 1 % of the best of all nine combinations of 1, 2 and 4 on average.
struct WaveKTile {
    int mi, ni;
    wavek_kernel_t fn[3];   // nullptr: not for this layout
};
#define AXONN_WAVEK(MI, NI) {gemm_wavek_kernel<true, false, MI, NI>, gemm_wavek_kernel<true, true, MI, NI>, gemm_wavek_kernel<false, false, MI, NI>}
static const WaveKTile kTiles[] = {
    {1, 1, AXONN_WAVEK(1, 1)},
    {1, 2, {gemm_wavek_kernel<true, false, 1, 2>, gemm_wavek_kernel<true, true, 1, 2>, nullptr}},
    {2, 2, AXONN_WAVEK(2, 2)},
    {2, 4, AXONN_WAVEK(2, 4)},
    {4, 4, AXONN_WAVEK(4, 4)},
};
#undef AXONN_WAVEK

// Modelled time of a launch in microseconds: launch, fill and drain, the adding up of partial tiles, plus the largest (smoothly) of
//   the chain of one wave:   its chunks, one after the other
//   a compute unit's work:   all chunks of the tiles it gets, its load path shared by its waves, and the
//                            exchange of partial tiles
//   memory:                  every operand and output byte once
//   staging:                 every byte that some tile loads, through the L2s
// Rows of an operand that do not start on 128-byte lines, or not on 16 bytes, make its loads touch more lines.
// Constants: least squares on the logarithm over 8 500 sampled products (1 to 16384 rows) on the four tiles and wave counts
// modelled shortest and two others each, the mean of operands in cache and from memory (residual 7-9 % near the best).  The smallest
// of some twenty estimates is an optimistic one: what is chosen takes 1.02 of it.
constexpr double kChosen = 1.02;
struct WaveKModel {
    double fill, chunk0, chunk_area, work_side, work_area, exchange, store, per_mb, staged_per_mb, off_line, off_piece, chain_lines, add_up;
};
static const WaveKModel kModel[3] = {
    {2.75, 0.205, 0.0289, 0.0245, 0.0, 0.260, 0.270, 0.224, 0.0308, 0.358, 0.147, 0.311, 0.79},      // NN
    {2.70, 0.178, 0.0345, 0.0188, 0.0021, 0.160, 0.406, 0.191, 0.0263, 0.399, 0.271, 0.299, 1.18},   // NT
    {3.01, 0.194, 0.0307, 0.0238, 0.0, 0.206, 0.235, 0.271, 0.0417, 0.274, 0.184, 0.340, 0.83},      // TN
};
// The figures of the rule for the scratch area (Figures::Area in axonn_linear.hip): they decide which plans use it and do not
// follow the kernel.
constexpr double kAreaChosen = 1.10;
static const WaveKModel kAreaModel[3] = {
    {4.0, 0.110, 0.045, 0.029, 0.0, 0.30, 0.20, 0.153, 0.044, 0.0, 0.0, 0.0, 0.0},       // NN
    {5.3, 0.141, 0.032, 0.010, 0.0076, 0.45, 0.14, 0.148, 0.038, 0.0, 0.0, 0.0, 0.0},    // NT
    {4.0, 0.105, 0.044, 0.033, 0.0, 0.31, 0.21, 0.153, 0.044, 0.0, 0.0, 0.0, 0.0},       // TN
};
static double model_us(const WaveKModel& m, int mi, int ni, int waves, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
    const double area = mi * ni, tiles = (double)((M + 16 * mi - 1) / (16 * mi)) * (double)((N + 16 * ni - 1) / (16 * ni));
    const int64_t n_chunks = (K + WaveKCfg::KC - 1) / WaveKCfg::KC;
    auto more_lines = [&](int64_t ld) { return (ld % 64 ? m.off_line : 0.0) + (ld % 8 ? m.off_piece : 0.0); };
    const double more = (more_lines(lda) * mi + more_lines(ldb) * ni) / (mi + ni);
    // Beyond one tile per compute unit a round more is a whole one: smoothed there as well, the model was 16-18 % short
    // just above 256, 512 and 768 tiles, and 2816 x 128 x 9856 TN went to 352 tiles of 32 x 32 (53.5 us) from split-K
    // (39.6).
    const double chunks = (double)n_chunks, full = tiles / 256.0;
    const double rounds = full > 1.0 ? std::ceil(full) : std::pow(1.0 + std::pow(full, 4.0), 0.25);
    const double chain = (double)((n_chunks + waves - 1) / waves) * (m.chunk0 + m.chunk_area * area) * (1.0 + m.chain_lines * more);
    const double unit = rounds * (chunks * (m.work_side * (mi + ni) * (1.0 + more) + m.work_area * area) +
                                  (waves > 1 ? m.exchange * waves * area / 16.0 : 0.0) + m.store * area / 16.0);
    const double memory = 2e-6 * ((double)M * K + (double)K * N + (double)M * N) * m.per_mb;
    const double staged = 2048e-6 * tiles * chunks * (mi + ni) * m.staged_per_mb * (1.0 + more);
    return m.fill + (waves > 1 ? m.add_up * area / 16.0 : 0.0) + std::cbrt(chain * chain * chain + unit * unit * unit + memory * memory * memory + staged * staged * staged);
}

WaveKChoice wavek_choose(int layout, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, bool area_rule) {
    const WaveKModel& model = (area_rule ? kAreaModel : kModel)[layout];
    WaveKChoice best;
    if (lda >= WaveKCfg::MAX_LD || ldb >= WaveKCfg::MAX_LD || (layout != 2 && K < 8)) return best;
    for (int i = 0; i < (int)(sizeof(kTiles) / sizeof(kTiles[0])); ++i) {
        const WaveKTile& t = kTiles[i];
        const int64_t tm = 16 * t.mi, tn = 16 * t.ni;
        if (!t.fn[layout]) continue;
        if (M < tm && (layout == 2 || t.mi > 2)) continue;   // see the kernel's requirements
        if (N < tn && (layout != 1 || t.ni > 2)) continue;
        if (t.mi * t.ni == 1 && ((layout != 1 && N >= 32) && (layout != 2 || M >= 32))) continue;   // narrow matrices only
        const int64_t tiles = ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
        for (int w = 1; w <= WaveKCfg::max_waves(t.mi, t.ni) && (w == 1 || (int64_t)(w - 1) * WaveKCfg::KC < K); w *= 2) {
            if (tiles * 64 * w >= ((int64_t)1 << 32)) continue;   // threads of a launch
            const double us = model_us(model, t.mi, t.ni, w, M, N, K, lda, ldb);
            if (best.tile < 0 || us < best.us) best = WaveKChoice{i, w, us};
        }
    }
    best.us *= area_rule ? kAreaChosen : kChosen;
    return best;
}

void wavek_tile(const WaveKChoice& c, int* rows, int* cols) {
    *rows = 16 * kTiles[c.tile].mi;
    *cols = 16 * kTiles[c.tile].ni;
}

// One wave over all of K on the 64 x 64 tile of two MN-contiguous operands: all of K is one chunk there.  900 sampled products on
// both kernels (1 to 64 k, 64 to 262144 rows, 64 to 20000 columns; operands in cache and from memory): below K = 64 gemm_shortk_kernel
// is 1.20 times as fast, but for 64 columns over more than 32 k, where one wave of a workgroup's four has work (65536 x 64 x 48
// 6.9 us against 5.5).  At K = 64 the wave-K kernel's k-rows are all there, and it is ahead (0.73 to 0.98 over narrow outputs, 0.90 to 0.95
// over rows off 128-byte lines, 9200 x 320 5.1 us against 6.4) until there are nine tiles a compute unit and more than 192 columns: from
// there whole lines run 1.13 times as fast on gemm_shortk_kernel, up to 512 columns off them 1.07 times, more columns off them 0.94.
// Outputs of more than 320 MB whose rows are no whole halves of a line: 42 products 0.87 times as fast on it (18336 x 21736 x 8 263 us and 178).
//
// Workgroups that write parts of one line run side by side behind one L2 (Chunks), where rows are no whole halves of a line: 1.06 to 1.10
// times as fast from 8 MB of output on (163 products); below, and for whole rows, up to 4 % slower.
ShortK wavek_short(const WaveKChoice& c, int layout, int64_t m, int64_t n, int64_t K, int64_t ldc) {
    if (layout != 2 || c.waves != 1 || kTiles[c.tile].mi != 4 || kTiles[c.tile].ni != 4 || K > 64) return ShortK::No;
    if (n % 32 != 0 && m * n > (int64_t)160 << 20) return ShortK::No;
    const bool ahead = K < 64 ? K <= 32 || n > 64 : n > 192 && (n % 64 == 0 || n <= 512) && (m + 63) / 64 * ((n + 63) / 64) >= 9 * 256;
    return !ahead ? ShortK::No : ldc % 32 != 0 && m * n >= (int64_t)4 << 20 ? ShortK::Chunks : ShortK::Yes;
}

static int lds_bytes(int tile, int waves, int layout) {
    return WaveKCfg::lds_bytes(layout != 2, layout == 1, kTiles[tile].mi, kTiles[tile].ni, waves);
}

void wavek_raise_lds_limit() {
    for (int i = 0; i < (int)(sizeof(kTiles) / sizeof(kTiles[0])); ++i)
        for (int l = 0; l < 3; ++l)
            if (kTiles[i].fn[l])
                (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kTiles[i].fn[l]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                          lds_bytes(i, WaveKCfg::max_waves(kTiles[i].mi, kTiles[i].ni), l));
}

void wavek_launch(const WaveKChoice& c, int layout, hipStream_t s, const uint16_t* A, const uint16_t* B, uint16_t* C,
                  int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc) {
    const WaveKTile& t = kTiles[c.tile];
    const ShortK short_k = wavek_short(c, layout, m, n, K, ldc);
    if (short_k != ShortK::No) {
        const int64_t tm = (m + 63) / 64, tn = (n + ShortKCfg::COLS - 1) / ShortKCfg::COLS;
        // from three workgroups a compute unit on, each takes two steps of columns: 3000 x 5000 x 24 8.9 -> 8.6 us, 8192 x 8192 x 40 33.9 ->
        // 28.7; 600 x 16384 x 7 (640 steps) 6.4 -> 6.9.  Four steps: 14 % slower on 2048 x 8192 x 24.
        const int64_t span = tm * tn >= 768 ? 2 : 1;
        const bool chunks = short_k == ShortK::Chunks;
        const auto kernel = K <= 32 ? (chunks ? gemm_shortk_kernel<1, true> : gemm_shortk_kernel<1, false>)
                                    : (chunks ? gemm_shortk_kernel<2, true> : gemm_shortk_kernel<2, false>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)(tm * ((tn + span - 1) / span))), dim3(256), 0, s,
                           A, B, C, m, n, (int)K, lda, ldb, ldc, (int)tn, (int)span);
        return;
    }
    const int64_t tiles_m = (m + 16 * t.mi - 1) / (16 * t.mi), tiles_n = (n + 16 * t.ni - 1) / (16 * t.ni);
    hipLaunchKernelGGL(t.fn[layout], dim3((unsigned)(tiles_m * tiles_n)), dim3(64 * c.waves), lds_bytes(c.tile, c.waves, layout), s,
                       A, B, C, m, n, K, lda, ldb, ldc, (int)tiles_m, (int)tiles_n, (int)(tiles_m < 8 ? tiles_m : 8));
}

}  // namespace axonn
