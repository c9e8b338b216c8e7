// Translation unit of the eight-wave tile kernels (see kernels.hpp).
#include "kernels.hpp"
#include "gemm_mfma16_k64g.hpp"

#include <algorithm>
#include <cmath>

namespace axonn {

// Modelled time of a launch in microseconds: launch, fill and drain, plus for every round of 256 workgroups the 64-k steps and
// what a tile costs beside them; a last round that fills a fraction f of the compute units counts last + (1 - last) f.  A step
// takes longer
//   as the operands outgrow the caches (16 MB and more: all of it): by `far`, and by `apart` times the share of a panel that the
//   tiles behind one L2 do not have in common (one tile column or row over the whole chip: half of it; a square patch: a fifth);
//   where the rows of an operand do not start on 128-byte lines: its loads then touch a line more (`lines`: of A K-contiguous, B
//   K-contiguous, A MN-contiguous, B MN-contiguous, times its share of the tile).  Where K-contiguous rows
//   are loaded by lines (GroupKLines) a step of theirs takes `late_line` longer (B) or no longer (A), and a tile `late` steps more: a stage
//   more is loaded and waited for.  (600 sampled products of K off 64, residual 7-11 %; what is chosen takes 1.004 times the best tile, 1.008
//   with the figures of the loads by k.)
// Outputs whose rows do not start on 128-byte lines pay for the lines that two workgroups write a part of.
// Least squares on the logarithm over 6 000 sampled products of up to 80 GFLOP, the mean of operands in cache and operands
// from memory, residual 5-8 %.  With the wave-K and the guarded kernel's models the choice is 0.8 % behind the best kernel measured
// on average, 5 % at the 95th percentile.  (96 x 128 and 192 x 128: 700 products of 48 to 900 tiles of 128 x 128, residual 4 %; they are
// chosen for a third of those, which then run 1.08 to 1.09 times as fast, the slowest 0.97; what is chosen takes 1.003 times the best tile, 1.032 without them.)
struct GroupTile {
    int bm, bn, groups, lds_bytes;
    double launch, tile, last, shared_lines, us64[3], far[3], apart[3], lines[4], late, late_line;
    tile_kernel_t fn[3], fn_tail[3];   // per layout; nullptr: not built
};
#define AXONN_GROUP3(BM, BN, G, ...) {gemm_tile_kernel_k64g<BM, BN, G, true, false, __VA_ARGS__>, gemm_tile_kernel_k64g<BM, BN, G, true, true, __VA_ARGS__>, \
                                      gemm_tile_kernel_k64g<BM, BN, G, false, false, __VA_ARGS__>}
// the 128 x 128 tile in two groups: where an operand is read with the transposing reads (K of 6000 and more, operands in cache:
// NN 3-7 % faster than one group, TN 8-11 %, NT +-1 %), and for whole K only
#define AXONN_GROUP2(BM, BN, G, ...) {gemm_tile_kernel_k64g<BM, BN, G, true, false, __VA_ARGS__>, nullptr, gemm_tile_kernel_k64g<BM, BN, G, false, false, __VA_ARGS__>}
#define AXONN_NO_KERNELS(...) {nullptr, nullptr, nullptr}
#define AXONN_GROUP_TILE(BM, BN, G, KERNELS, TAIL_KERNELS, ...) {BM, BN, G, group_lds<BM, BN, G>(), __VA_ARGS__, KERNELS(BM, BN, G, false), TAIL_KERNELS(BM, BN, G, true)}
static const GroupTile kTiles[] = {
    AXONN_GROUP_TILE(64, 64, 2, AXONN_GROUP3, AXONN_GROUP3, 3.04, 0.48, 0.770, 0.09, {0.141, 0.124, 0.155}, {0.073, 0.131, 0.0}, {2.118, 2.712, 1.544}, {0.44, 0.51, 0.49, 0.60}, 1.8, 0.06),
    AXONN_GROUP_TILE(64, 128, 1, AXONN_GROUP3, AXONN_GROUP3, 2.22, 1.33, 0.789, 0.21, {0.229, 0.202, 0.258}, {0.209, 0.349, 0.036}, {1.099, 1.396, 1.135}, {0.47, 0.49, 0.35, 0.30}, 2.4, 0.03),
    AXONN_GROUP_TILE(128, 64, 1, AXONN_GROUP3, AXONN_GROUP3, 2.25, 1.28, 0.814, 0.26, {0.224, 0.201, 0.255}, {0.314, 0.421, 0.130}, {0.791, 0.978, 0.611}, {0.43, 0.56, 0.19, 0.64}, 2.6, 0.06),
    AXONN_GROUP_TILE(96, 128, 1, AXONN_GROUP3, AXONN_GROUP3, 2.51, 0.99, 0.871, 0.37, {0.355, 0.342, 0.392}, {0.036, 0.080, 0.0}, {0.519, 0.539, 0.624}, {0.17, 0.29, 0.05, 0.27}, 1.3, 0.01),
    AXONN_GROUP_TILE(192, 128, 1, AXONN_GROUP3, AXONN_GROUP3, 1.98, 1.99, 0.794, 1.70, {0.563, 0.529, 0.604}, {0.028, 0.086, 0.0}, {0.431, 0.312, 0.245}, {0.19, 0.56, 0.06, 0.31}, 0.0, 0.0),
    AXONN_GROUP_TILE(128, 128, 1, AXONN_GROUP3, AXONN_GROUP3, 2.16, 1.82, 0.812, 1.04, {0.338, 0.308, 0.408}, {0.276, 0.381, 0.112}, {0.509, 0.583, 0.290}, {0.36, 0.44, 0.11, 0.21}, 1.8, 0.04),
    AXONN_GROUP_TILE(128, 128, 2, AXONN_GROUP2, AXONN_NO_KERNELS, 2.51, 2.69, 0.806, 0.96, {0.311, 0.0, 0.341}, {0.299, 0.0, 0.159}, {0.665, 0.0, 0.579}, {0.42, 0.44, 0.22, 0.26}, 0.0, 0.0),
    AXONN_GROUP_TILE(256, 128, 1, AXONN_GROUP3, AXONN_GROUP3, 1.93, 3.34, 0.693, 3.57, {0.609, 0.598, 0.728}, {0.130, 0.155, 0.0}, {0.472, 0.557, 0.260}, {0.32, 0.30, 0.03, 0.23}, 0.0, 0.0),
    // (NN and NT step: 0.635 and 0.581 fitted.  Near a tie of the half tiles this one is taken.  NT: 1.4 % ahead with operands from memory, 0.4 %
    // in cache, nine products.  NN: 2.2 % ahead from memory, 1.5-4.5 % behind in cache, the 70 sampled products that the figure decides.)
    AXONN_GROUP_TILE(128, 256, 1, AXONN_GROUP3, AXONN_GROUP3, 1.86, 3.41, 0.692, 2.91, {0.612, 0.562, 0.716}, {0.071, 0.155, 0.0}, {0.760, 0.848, 0.358}, {0.13, 0.43, 0.06, 0.10}, 0.0, 0.0),
};
#undef AXONN_GROUP_TILE
#undef AXONN_GROUP3
#undef AXONN_GROUP2
#undef AXONN_NO_KERNELS

static const GroupTile* find(int bm, int bn, int groups) {
    for (const GroupTile& t : kTiles)
        if (t.bm == bm && t.bn == bn && t.groups == groups) return &t;
    return nullptr;
}

tile_kernel_t group_kernel(int bm, int bn, int groups, int layout, bool k_tail) {
    const GroupTile* t = find(bm, bn, groups);
    return t ? (k_tail ? t->fn_tail : t->fn)[layout] : nullptr;
}

int group_lds_bytes(int bm, int bn, int groups) {
    const GroupTile* t = find(bm, bn, groups);
    return t ? t->lds_bytes : 0;
}

static double model_us(const GroupTile& t, int layout, int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc) {
    if (!(K % 64 ? t.fn_tail : t.fn)[layout] || m < t.bm || n < t.bn || K <= 64) return -1.0;
    const int64_t wgs = ((m + t.bm - 1) / t.bm) * ((n + t.bn - 1) / t.bn), rest = wgs % 256;
    const double rounds = (double)(wgs / 256) + (rest ? t.last + (1.0 - t.last) * (double)rest / 256.0 : 0.0);
    const bool late = K % 64 && K > kGroupLinesK && group_lines(t.bm, t.bn, layout != 2, layout == 1);
    const double line_a = layout == 2 ? t.lines[2] : late ? 0.0 : t.lines[0], line_b = layout != 1 ? t.lines[3] : late ? t.late_line : t.lines[1];
    const double lines = 1.0 + (lda % 64 ? line_a * t.bm / (t.bm + t.bn) : 0.0) + (ldb % 64 ? line_b * t.bn / (t.bm + t.bn) : 0.0);
    const double shared = ldc % 64 == 0 ? 0.0 : ldc % 32 == 0 ? 0.15 : 1.0;
    const double full = (double)wgs / 256.0 - 0.5;
    const double mb = 2e-6 * ((double)m * K + (double)K * n);
    // the up to 32 tiles that run behind one L2 are up to eight tile rows high (map_workgroup)
    const double tiles_m = (double)((m + t.bm - 1) / t.bm), behind = std::min(std::ceil((double)wgs / 8.0), 32.0);
    const double rows = std::min(std::min(tiles_m, 8.0), behind), cols = std::ceil(behind / rows);
    const double panels = (rows * t.bm + cols * t.bn) / (behind * (t.bm + t.bn));
    const double step = t.us64[layout] * lines * (1.0 + (t.far[layout] + t.apart[layout] * panels) * std::min(1.0, mb / 16.0));
    const double steps = (double)((K + 63) / 64) + (late ? t.late : 0.0);
    return t.launch + rounds * (steps * step + t.tile) + (full > 0.0 ? shared * t.shared_lines * full : 0.0);
}

double group_us(int bm, int bn, int groups, int layout, int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc) {
    const GroupTile* t = find(bm, bn, groups);
    return t ? model_us(*t, layout, m, n, K, lda, ldb, ldc) : -1.0;
}

// Tiles of 96 and 192 rows: by how much more than modelled they count; < 0: not there.  Within the range that the model was fitted over.  Beyond a round of workgroups over a short K it is 5 to
// 13 % short (9344 x 9344 x 384 TN 73 us on 256 x 256 tiles, 83 here; 1920 x 12416 x 512 27 and 29, 1536 x 6272 x 640 16.4 and 17.1; in one round
// 1280 x 3712 x 384 TN 8.2 us on 256 x 128 and 7.3 here).
// TN in more than one round: not there.  256 x 256 tiles read an eighth less in their two rounds (23 such products: 0.988 here, 1152 x 7680 x 1152 26.2 us
// there and 27.6 here), while in one round 62 TN products run 1.07 to 1.14 times as fast.
// Rows of the output off 128-byte lines make no difference in one round: 750 products that go to these tiles by up to 15 % of modelled time run 1.06 (NN),
// 1.10 (NT) and 1.07 (TN) times as fast here, 1.03 to 1.08 those within 2 % of a tie (1064 x 4168 x 1608 NT 26.4 us on 128 x 256 tiles, 22.2 on 192 x 128).
// In NT beyond a round 192 x 128 has to be 15 % ahead there: eleven such products on 256 x 256 tiles run 1.06 times as fast here with operands in
// cache and 0.91 times from memory (3859 x 2888 x 5760 124 and 116 us, from memory 111 and 123).
static double between_margin(const GroupTile& t, int layout, int64_t m, int64_t n, int64_t K, int64_t ldc) {
    const int64_t wgs = ((m + t.bm - 1) / t.bm) * ((n + t.bn - 1) / t.bn);
    if (K < 320 || (wgs > 256 && (K < 640 || layout == 2)) || m * n > (int64_t)16 << 20) return -1.0;
    return wgs > 256 && layout == 1 && t.bm == 192 && ldc % 64 != 0 ? 1.15 : 1.0;
}

GroupChoice group_choose(int layout, int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc) {
    GroupChoice best;
    for (int i = 0; i < (int)(sizeof(kTiles) / sizeof(kTiles[0])); ++i) {
        const GroupTile& t = kTiles[i];
        if (t.groups == 1 && t.bm % 128 == 0 && t.bn % 128 == 0) continue;   // variants of their own
        const double margin = t.bm % 96 == 0 ? between_margin(t, layout, m, n, K, ldc) : 1.0;
        const double us = margin * model_us(t, layout, m, n, K, lda, ldb, ldc);
        if (margin > 0.0 && us >= 0.0 && (best.tile < 0 || us < best.us)) best = GroupChoice{i, us};
    }
    return best;
}

void group_tile(const GroupChoice& c, int* rows, int* cols, int* groups) {
    *rows = kTiles[c.tile].bm;
    *cols = kTiles[c.tile].bn;
    *groups = kTiles[c.tile].groups;
}

void group_launch(const GroupChoice& c, int layout, hipStream_t s, const uint16_t* A, const uint16_t* B, uint16_t* C,
                  int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc) {
    const GroupTile& t = kTiles[c.tile];
    const int tiles_m = (int)((m + t.bm - 1) / t.bm), tiles_n = (int)((n + t.bn - 1) / t.bn), k_tail = (int)(K % 64);
    hipLaunchKernelGGL(k_tail ? t.fn_tail[layout] : t.fn[layout], dim3((unsigned)((int64_t)tiles_m * tiles_n)), dim3(512), t.lds_bytes, s, A, B, C,
                       (int)(K - k_tail + (k_tail ? 64 : 0)), (int)lda, (int)ldb, (int)ldc,
                       TileGrid{tiles_m, tiles_n, (int)(m - t.bm), (int)(n - t.bn), k_tail}, tiles_m < 8 ? tiles_m : 8, SplitK{});
}

// ---- split-K ----------------------------------------------------------------------------------------------------------------------
// Modelled time: launch and exchange, plus for every round of 256 workgroups the 64-k steps of a range and what it costs beside them,
// plus the bytes of partial sums that are written and read back (`moved`, per MB).  Least squares over 700 sampled products that are planned
// with split-K, operands in cache, of three sets in turn, and from memory (residual 7-10 %); what is chosen takes 1.011 times the best of the
// tiles and counts measured.
struct GroupSplitTile {
    int bm, bn, lds_bytes;
    double launch, us64[3], apart, tile, moved, last;
    void (*fn[3])(const uint16_t*, const uint16_t*, uint16_t*, int, int, int, int, int, int, int, GroupSplit);
};
#define AXONN_SPLIT_TILE(BM, BN, ...) {BM, BN, GroupCfg<BM, BN, 1>::LDS_BYTES, __VA_ARGS__, {gemm_tile_kernel_k64gs<BM, BN, true, false>, \
                                       gemm_tile_kernel_k64gs<BM, BN, true, true>, gemm_tile_kernel_k64gs<BM, BN, false, false>}}
static const GroupSplitTile kSplitTiles[] = {
    AXONN_SPLIT_TILE(64, 128, 7.27, {0.203, 0.203, 0.213}, 1.263, 7.02, 0.317, 0.800),
    AXONN_SPLIT_TILE(128, 128, 7.71, {0.376, 0.376, 0.381}, 0.577, 7.66, 0.365, 0.672),
    AXONN_SPLIT_TILE(256, 128, 6.27, {0.561, 0.556, 0.548}, 0.865, 10.0, 0.792, 0.594),
    AXONN_SPLIT_TILE(128, 256, 8.87, {0.690, 0.708, 0.722}, 0.0, 7.91, 0.556, 0.764),
};
#undef AXONN_SPLIT_TILE
static const int kSplitCounts[] = {2, 3, 4, 5, 6, 8};   // the ones that group_tile has an exchange for

size_t group_split_bytes(const GroupSplitChoice& c, int64_t m, int64_t n) {
    return c.tile < 0 ? 0 : (size_t)(m * n * c.splits) * sizeof(float);   // whole tiles
}

GroupSplitChoice group_split_choose(int layout, int64_t m, int64_t n, int64_t K, size_t max_bytes, int64_t max_flags) {
    GroupSplitChoice best;
    if (K % 64 != 0) return best;
    for (int i = 0; i < (int)(sizeof(kSplitTiles) / sizeof(kSplitTiles[0])); ++i) {
        const GroupSplitTile& t = kSplitTiles[i];
        if (m % t.bm != 0 || n % t.bn != 0) continue;
        const int64_t tiles_m = m / t.bm, tiles = tiles_m * (n / t.bn);
        for (const int splits : kSplitCounts) {
            const int64_t wgs = tiles * splits, rest = wgs % 256;
            // up to two rounds: more were not tried
            if (wgs > 512 || K / 64 < splits || tiles * splits * (splits - 1) > max_flags) continue;
            if (group_split_bytes(GroupSplitChoice{i, splits, 0.0}, m, n) > max_bytes) continue;
            // the ranges of a tile run behind one L2, each over another K: fewer tiles there have a panel in common
            const double behind = std::max(std::min(std::ceil((double)wgs / 8.0), 32.0) / splits, 1.0);
            const double rows = std::min(std::min((double)tiles_m, 8.0), behind), cols = std::max(behind / rows, 1.0);
            const double panels = (rows * t.bm + cols * t.bn) / (behind * (t.bm + t.bn));
            const double step = t.us64[layout] * (1.0 + t.apart * panels * std::min(1.0, 2e-6 * (double)K * (double)(m + n) / 16.0));
            const double rounds = (double)(wgs / 256) + (rest ? t.last + (1.0 - t.last) * (double)rest / 256.0 : 0.0);
            const double moved = 8e-6 * (double)m * (double)n * (splits - 1) / splits;
            const double us = t.launch + rounds * ((double)((K / 64 + splits - 1) / splits) * step + t.tile) + t.moved * moved;
            if (best.tile < 0 || us < best.us) best = GroupSplitChoice{i, splits, us};
        }
    }
    return best;
}

void group_split_tile(const GroupSplitChoice& c, int* rows, int* cols) {
    *rows = kSplitTiles[c.tile].bm;
    *cols = kSplitTiles[c.tile].bn;
}

void group_split_launch(const GroupSplitChoice& c, int layout, hipStream_t s, const uint16_t* A, const uint16_t* B, uint16_t* C, int64_t m, int64_t n,
                        int64_t K, int64_t lda, int64_t ldb, int64_t ldc, float* partials, uint32_t* flags, uint32_t epoch, uint32_t probes) {
    const GroupSplitTile& t = kSplitTiles[c.tile];
    const int tiles_m = (int)(m / t.bm), tiles_n = (int)(n / t.bn);
    hipLaunchKernelGGL(t.fn[layout], dim3((unsigned)(tiles_m * tiles_n * c.splits)), dim3(512), t.lds_bytes, s, A, B, C, (int)K, (int)lda, (int)ldb, (int)ldc,
                       tiles_m, tiles_n, tiles_m < 8 ? tiles_m : 8, GroupSplit{partials, flags, epoch, probes, c.splits});
}

void group_raise_lds_limit() {
    for (const GroupTile& t : kTiles)
        for (int l = 0; l < 3; ++l)
            for (const tile_kernel_t fn : {t.fn[l], t.fn_tail[l]})
                if (fn) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, t.lds_bytes);
    for (const GroupSplitTile& t : kSplitTiles)
        for (const auto fn : t.fn) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, t.lds_bytes);
}

}  // namespace axonn
