// Re-storing a bf16 operand for another GEMM mode (paper Sec. IV-C: NN, NT and TN differ only in how
// each operand lies in memory): dst[c * rows + r] = src[r * cols + c], 16-bit elements, bits moved.
//
// HBM-bound: 2 bytes read and 2 bytes written per element, nothing else.  The tile kernel moves a
// 64 x 64 tile per workgroup: 16-byte global loads of whole 128-byte row segments into LDS (row
// stride 144 bytes, which keeps the reads below conflict-free), then the transposing LDS read
// ds_read_b64_tr_b16 -- a 16-lane group turns a 4-row x 16-column block into, per lane, one column's
// four consecutive rows -- twice per lane for eight consecutive rows, i.e. 16 bytes of one output
// row, stored with one 16-byte global store.  A wave writes 16 output rows x 64 bytes per store and
// the two stores of a wave complete each 128-byte line.
//
// Any size of at least a tile: the last tiles are moved back to the matrix' edge (what they repeat is stored
// twice, the same bits), and loads and stores take any 2-byte aligned address.  One element per thread, as
// before, 2049 x 4100 took 29 us; now 16 (floor at the rate of a large copy: 6.5; the rest is lines that two tiles
// write a part of).
//
// Order of the tiles.  Row by row for whole tiles.  BANDS, for large matrices whose rows are no whole lines or whose
// both strides are multiples of 4 KB: each XCD works on a contiguous chunk of the tiles, four deep along the
// shorter side of the matrix (with output rows that are no whole lines but whole 16-byte pieces: always along those; 3000 x
// 9000 from HBM 34 -> 30 us), and each such band starts 5 tiles further along.  In the first case two tiles
// that write parts of one line then do it behind the same L2 (2049 x 4100 from HBM 19 -> 16 us); in the second, the
// lines of a tile fall on few memory channels, and it is the neighbouring tiles that use the others (from HBM:
// 4096 x 12288 50 -> 43 us, 8192 x 8192 67 -> 53, 4096 x 16384 66 -> 53; floors 39, 52, 52).  Anywhere else it is 3-10 % behind
// (3136 x 15872 47.6 -> 50.0, 11904 x 1280 16.4 -> 18.3), and below 1024 tiles, which all fit the chip side by side, its
// index arithmetic costs 0.4 us of 3.  Tiles of 64 x 128, 128 x 64 and 128 x 128 were no faster; non-temporal stores 5 % faster
// from 128 MB on, slower below, and half as fast where rows are not whole lines.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace axonn {

typedef uint32_t tr_u32x4 __attribute__((ext_vector_type(4)));
typedef tr_u32x4 __attribute__((aligned(2))) tr_u32x4_any;   // at any 2-byte aligned address
typedef short tr_v4i16 __attribute__((ext_vector_type(4)));

constexpr int TR_TILE = 64;          // rows and columns per workgroup
constexpr int TR_BAND = 4;           // tiles across a band
inline bool tr_bands(int64_t rows, int64_t cols, int64_t tiles, bool whole) {
    return tiles >= 1024 && (!whole || (rows % 2048 == 0 && cols % 2048 == 0));
}
// A ragged matrix takes the tile kernel from this many elements on: below, the launch is all that counts, and a
// narrow one still gives the element kernel the more workgroups (4589 x 193: 3.6 us against 4.2; 1000 x 1000: 4.0
// against 3.0).
constexpr int64_t tr_ragged_from(int64_t narrow) { return narrow < 256 ? 3 << 19 : 1 << 18; }
inline int64_t tr_tiles(int64_t extent) { return (extent + TR_TILE - 1) / TR_TILE; }
enum class TrKernel { Refused, Element, Tile, TileBands };
// `aligned`: both pointers on 16-byte boundaries.
inline TrKernel tr_choose(int64_t rows, int64_t cols, bool aligned) {
    const bool whole = rows % TR_TILE == 0 && cols % TR_TILE == 0 && aligned;
    if (!whole && (cols + 3) / 4 > 65535) return TrKernel::Refused;   // the element kernel's grid, whichever kernel runs
    const int64_t tiles = tr_tiles(rows) * tr_tiles(cols);
    // 256 threads a tile, and a launch holds fewer than 2^32 in one dimension: the element kernel has two
    const bool ragged_tiles = std::min(rows, cols) >= TR_TILE && rows * cols >= tr_ragged_from(std::min(rows, cols)) && tiles < ((int64_t)1 << 24);
    if (!whole && !ragged_tiles) return TrKernel::Element;
    return tr_bands(rows, cols, tiles, whole) ? TrKernel::TileBands : TrKernel::Tile;
}
constexpr int TR_LDS_STRIDE = 144;   // bytes per tile row in LDS (128 + 16)

// Requires rows >= 64, cols >= 64.  grid = tiles, block = 256.
template <bool BANDS>
__global__ __launch_bounds__(256) void transpose_tile_kernel(const uint16_t* __restrict__ src,
                                                             uint16_t* __restrict__ dst, int64_t rows,
                                                             int64_t cols, int tiles_r, int tiles_c) {
    __shared__ __attribute__((aligned(16))) uint8_t tile[TR_TILE * TR_LDS_STRIDE];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint32_t tr, tc;
    if constexpr (BANDS) {
        // XCD x runs the workgroups x, x + 8, ...: a contiguous chunk of the sequence
        const uint32_t x = blockIdx.x & 7, rem = gridDim.x & 7;
        const uint32_t id = x * (gridDim.x >> 3) + min(x, rem) + (blockIdx.x >> 3);
        const bool tall = tiles_r > tiles_c || ((rows & (TR_TILE - 1)) && !(rows & 7));   // bands of four tile columns, else of four tile rows
        const uint32_t across = tall ? tiles_c : tiles_r, along = tall ? tiles_r : tiles_c;
        const uint32_t band = id / (TR_BAND * along), in_band = id - band * (TR_BAND * along);
        const uint32_t depth = min(across - band * TR_BAND, (uint32_t)TR_BAND);
        const uint32_t in_line = in_band / depth;
        const uint32_t a = band * TR_BAND + in_band - in_line * depth, l = (in_line + band * 5) % along;
        tr = tall ? l : a;
        tc = tall ? a : l;
    } else {
        tr = blockIdx.x / (uint32_t)tiles_c;
        tc = blockIdx.x - tr * tiles_c;
    }
    const int64_t r0 = min((int64_t)tr * TR_TILE, rows - TR_TILE), c0 = min((int64_t)tc * TR_TILE, cols - TR_TILE);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int q = t + 256 * u, row = q >> 3, ch = q & 7;   // 16-byte chunk ch of tile row `row`
        const tr_u32x4 v = *reinterpret_cast<const tr_u32x4_any*>(src + (r0 + row) * cols + c0 + ch * 8);
        *reinterpret_cast<tr_u32x4*>(tile + row * TR_LDS_STRIDE + ch * 16) = v;
    }
    __syncthreads();
    // wave w owns tile columns 16w .. 16w+15 (16 output rows); lane = 16 g + s
    const int g = lane >> 4, s = lane & 15;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        // the group reads tile rows rb*32 + 8g + 0..3 (then + 4..7); lane s supplies row s>>2,
        // columns 16w + 4*(s&3) .. +3, and receives column 16w + s
        const uint8_t* p = tile + (rb * 32 + 8 * g + (s >> 2)) * TR_LDS_STRIDE + (16 * wave + 4 * (s & 3)) * 2;
        typedef __attribute__((address_space(3))) tr_v4i16 lds_v4i16;
        const tr_v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(p));
        const tr_v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(p + 4 * TR_LDS_STRIDE));
        tr_u32x4 out;
        out[0] = __builtin_bit_cast(uint32_t, __builtin_shufflevector(lo, lo, 0, 1));
        out[1] = __builtin_bit_cast(uint32_t, __builtin_shufflevector(lo, lo, 2, 3));
        out[2] = __builtin_bit_cast(uint32_t, __builtin_shufflevector(hi, hi, 0, 1));
        out[3] = __builtin_bit_cast(uint32_t, __builtin_shufflevector(hi, hi, 2, 3));
        *reinterpret_cast<tr_u32x4_any*>(dst + (c0 + 16 * wave + s) * rows + r0 + rb * 32 + 8 * g) = out;
    }
}

// Any rows, cols >= 1 (used below a tile in either direction and for small ragged matrices): one element per thread, stores coalesced along
// the output rows.
__global__ __launch_bounds__(256) void transpose_naive_kernel(const uint16_t* __restrict__ src,
                                                              uint16_t* __restrict__ dst, int64_t rows,
                                                              int64_t cols) {
    const int64_t r = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const int64_t c = (int64_t)blockIdx.y * 4 + (threadIdx.x >> 6);
    if (r < rows && c < cols) dst[c * rows + r] = src[r * cols + c];
}

}  // namespace axonn
