// The GEMM kernels are compiled in several translation units (the compile time is theirs); this
// header is what the host side (axonn_linear.hip) sees of them: one look-up function per unit.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_mfma.hpp"

namespace axonn {

// (A, B, C, K, lda, ldb, ldc, tiles, group_m, split-K state): leading dimensions in elements of
// the operands as stored, so that a launch can cover a block of rows or columns of a larger product
typedef void (*tile_kernel_t)(const uint16_t*, const uint16_t*, uint16_t*, int, int, int, int, TileGrid, int, SplitK);

// layout: 0 NN, 1 NT, 2 TN.  k_tail: the form for a K that is no multiple of 64 (TileGrid).  nullptr: no such kernel.
// 32-k LDS ring (gemm_tile_kernel16): tile bm x bn
tile_kernel_t ring_kernel_large(bool split, int layout);                          // 2 x 4 waves, with or without split-K: 256x256
tile_kernel_t ring_kernel_small(int bm, int bn, int layout);                       // 2 x 2 waves, split-K: 256x128, 128x256, 128x128 (not NT)
// 64-k stages (gemm_tile_kernel_k64): 256 x 256, 2 x 4 waves
tile_kernel_t k64_kernel(bool split, int layout, bool k_tail = false);
// the same on 256 x 128, 128 x 256 and 128 x 128 tiles, 2 x 2 waves, three LDS buffers per operand (NT with split-K only)
tile_kernel_t k64_kernel_half(int bm, int bn, int layout);
// the same with one resident workgroup per compute unit walking a list of tiles (gemm_tile_kernel_k64p)
tile_kernel_t k64p_kernel(int layout);

// Where the eight-wave kernel loads the K-contiguous operands of a K that is no multiple of 64 by lines (GroupKLines): beyond this K.  Up to there
// the stage more and the prologue cost what the lines save (operands in cache, from memory: 0.96 and 1.00 of the speed of the loads by k over
// K of 256 to 520, 0.97 and 1.05 over 520 to 800; from 1000 on 1.01 and 1.12, from 2500 on 1.27 and 1.25).
constexpr int kGroupLinesK = 768;

// eight waves on tiles from 64 x 64 to 256 x 128 (gemm_tile_kernel_k64g), no split-K
tile_kernel_t group_kernel(int bm, int bn, int groups, int layout, bool k_tail);
int group_lds_bytes(int bm, int bn, int groups);
double group_us(int bm, int bn, int groups, int layout, int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc);   // modelled time; < 0: not there
void group_raise_lds_limit();
// the tiles that are no variants: 64 x 64, 64 x 128, 128 x 64, 96 x 128, 192 x 128, and 128 x 128 in two groups
struct GroupChoice {
    int tile = -1;              // < 0: none of them takes this block
    double us = 0.0;            // modelled time
};
GroupChoice group_choose(int layout, int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc);
void group_tile(const GroupChoice& c, int* rows, int* cols, int* groups);
void group_launch(const GroupChoice& c, int layout, hipStream_t s, const uint16_t* A, const uint16_t* B, uint16_t* C,
                  int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc);

// the same kernel in several K ranges per tile (gemm_tile_kernel_k64gs), for blocks of whole tiles; through the scratch area
struct GroupSplitChoice {
    int tile = -1, splits = 0;  // tile < 0: none takes this block within the limits
    double us = 0.0;            // modelled time
};
GroupSplitChoice group_split_choose(int layout, int64_t m, int64_t n, int64_t K, size_t max_bytes, int64_t max_flags);
size_t group_split_bytes(const GroupSplitChoice& c, int64_t m, int64_t n);   // of partial sums
void group_split_tile(const GroupSplitChoice& c, int* rows, int* cols);
// How often a range looks again for the others of its tile before it hands its share on (split_exchange.hpp), about a microsecond each.  63 products of
// 11 to 300 us on an idle chip, against looking for ever: 0 times 1.136 of the time, 8 1.060, 32 1.006, 64 and 256 1.000.
constexpr uint32_t kGroupSplitProbes = 256;
// epoch: neither 0 nor ~0, another one for every launch
void group_split_launch(const GroupSplitChoice& c, int layout, hipStream_t s, const uint16_t* A, const uint16_t* B, uint16_t* C, int64_t m, int64_t n,
                        int64_t K, int64_t lda, int64_t ldb, int64_t ldc, float* partials, uint32_t* flags, uint32_t epoch, uint32_t probes);

// guarded MFMA kernel (gemm_edge_kernel): any m, n, K >= 1 and any leading dimensions
void edge_kernel_raise_lds_limit();
void edge_kernel_launch(int layout, unsigned workgroups, hipStream_t s, const uint16_t* A, const uint16_t* B, uint16_t* C,
                        int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc, int tiles_n);

// wave-K kernel (gemm_wavek_kernel): few tiles, few rows, rows at any address; a tile split over the waves of a workgroup
struct WaveKChoice {
    int tile = -1, waves = 0;   // tile < 0: the kernel does not take this block
    double us = 0.0;            // modelled time
};
// area_rule: by the figures that decide which plans use the scratch area
WaveKChoice wavek_choose(int layout, int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, bool area_rule = false);
void wavek_tile(const WaveKChoice& c, int* rows, int* cols);   // of its output tile
enum class ShortK { No, Yes, Chunks };   // whether it runs on gemm_shortk_kernel, and in which order of its workgroups
ShortK wavek_short(const WaveKChoice& c, int layout, int64_t m, int64_t n, int64_t K, int64_t ldc);
void wavek_raise_lds_limit();
void wavek_launch(const WaveKChoice& c, int layout, hipStream_t s, const uint16_t* A, const uint16_t* B, uint16_t* C,
                  int64_t m, int64_t n, int64_t K, int64_t lda, int64_t ldb, int64_t ldc);

}  // namespace axonn
