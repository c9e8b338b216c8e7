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
// before, 2049 x 4100 took 29 us; on this kernel 16 (floor at the rate of a large copy: 6.5; the rest is lines that two
// tiles write a part of: see transpose_window_kernel).
//
// Order of the tiles.  Row by row for whole tiles.  BANDS, for large matrices whose rows are no whole lines or whose
// both strides are multiples of 4 KB: each XCD works on a contiguous chunk of the tiles, four deep along the
// shorter side of the matrix (with output rows that are no whole lines but whole 16-byte pieces: always along those, 3-10 %), and each such band starts 5 tiles further along.  In the first case two tiles
// that write parts of one line then do it behind the same L2 (2049 x 4100 from HBM 19 -> 16 us; matrices of that size have gone to transpose_window_kernel since); in the second, the
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
// transpose_window_kernel: output elements along an output row per workgroup, threads, tile columns across a band
constexpr int TR_WINDOW = 128;
constexpr int TR_WINDOW_THREADS = 512;
constexpr int TR_WINDOW_BAND = 8;
constexpr int TR_WINDOW_STRIDE = 33;          // dwords per src row in LDS
inline int64_t tr_windows(int64_t rows) { return (rows + 63 + TR_WINDOW - 1) / TR_WINDOW; }   // a window starts up to 63 early
inline bool tr_bands(int64_t rows, int64_t cols, int64_t tiles, bool whole) {
    return tiles >= 1024 && (!whole || (rows % 2048 == 0 && cols % 2048 == 0));
}
// A ragged matrix takes the tile kernel from this many elements on: below, the launch is all that counts, and a
// narrow one still gives the element kernel the more workgroups (4589 x 193: 3.6 us against 4.2; 1000 x 1000: 4.0
// against 3.0).
constexpr int64_t tr_ragged_from(int64_t narrow) { return narrow < 256 ? 3 << 19 : 1 << 18; }
inline int64_t tr_tiles(int64_t extent) { return (extent + TR_TILE - 1) / TR_TILE; }
enum class TrKernel { Refused, Element, Tile, TileBands, Window };
// Whether the tile kernels leave a matrix to transpose_window_kernel.  Where output rows start at odd addresses it is ahead from
// some 600 tiles on (1001 x 3000, 752 tiles: 4.8 -> 4.2 us; 1001 x 2000, 512 tiles: 3.3 -> 3.7); where at even ones, from some 2500
// on (2008 x 5000, 2528 tiles: 7.8 -> 7.5 us; 1608 x 4168, 1716 tiles: 5.4 -> 5.9).
// A launch of 512 threads per window and tile column holds fewer than 2^32.
inline bool tr_window(int64_t rows, int64_t cols, uintptr_t dst) {
    if ((rows % 64 == 0 && dst % 128 == 0) || tr_windows(rows) * tr_tiles(cols) >= ((int64_t)1 << 23)) return false;
    return tr_tiles(rows) * tr_tiles(cols) >= ((rows % 2 || dst % 4) ? 640 : 2560);
}
// The one decision on a matrix: what is launched and what is told of it.
inline TrKernel tr_choose(int64_t rows, int64_t cols, uintptr_t src, uintptr_t dst) {
    const bool whole = rows % TR_TILE == 0 && cols % TR_TILE == 0 && ((src | dst) & 15) == 0;
    if (!whole && (cols + 3) / 4 > 65535) return TrKernel::Refused;   // the element kernel's grid, whichever kernel runs
    const int64_t tiles = tr_tiles(rows) * tr_tiles(cols);
    // 256 threads a tile, and a launch holds fewer than 2^32 in one dimension: the element kernel has two
    const bool ragged_tiles = std::min(rows, cols) >= TR_TILE && rows * cols >= tr_ragged_from(std::min(rows, cols)) && tiles < ((int64_t)1 << 24);
    if (!whole && !ragged_tiles) return TrKernel::Element;
    if (tr_window(rows, cols, dst)) return TrKernel::Window;
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

// Output rows that do not start on 128-byte lines (rows no multiple of 64, or dst off a line): the stores of a 64 x 64 tile
// end in lines that another tile writes the rest of, and at odd addresses each is several accesses.  Here the window of a
// workgroup follows the lines: of output row c it writes TR_WINDOW elements from the line boundary at or before r0 on, so
// that every store is an aligned 16-byte piece and a wave's store eight whole lines; only the first and last pieces of an
// output row go element by element.  The window starts up to 63 elements earlier from one output row to the next, so a
// workgroup reads TR_WINDOW + 63 rows of src (the compute units of an XCD work on a band of tiles side by side, and what
// two of them read comes from its L2).  The shift differs per output row, so the transposing LDS read does not fit; 16-bit reads
// from rows of an odd number of dwords do, spread over the banks.
// us, operands in cache / from HBM: 2049 x 4100 12.4 / 15.4 -> 7.1 / 10.7 (as a copy: 6.5), 8191 x 8193 72 / 87 -> 42 / 56,
// 701 x 9001 8.2 / 10.3 -> 6.0 / 8.4, 4104 x 4104 12.5 / 18.9 -> 11.7 / 16.9.  Windows of 192 elements: 2-8 % slower up to
// 2000 tiles, level above; 256: 10 %; 192 on four waves: another 5 %; 448: 20 %.  Bands of 4 or 16: +-3 %.
// Requires rows >= 1, cols >= 64.  grid = tr_windows(rows) x tr_tiles(cols).
__global__ __launch_bounds__(TR_WINDOW_THREADS) void transpose_window_kernel(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, int64_t rows,
                                                               int64_t cols, int tiles_r, int tiles_c) {
    constexpr int NT = TR_WINDOW_THREADS, IN_ROWS = TR_WINDOW + 64;
    __shared__ uint32_t tile[IN_ROWS * TR_WINDOW_STRIDE];
    const int t = threadIdx.x;
    // XCD x runs the workgroups x, x + 8, ...: a contiguous chunk of the sequence
    const uint32_t x = blockIdx.x & 7, rem = gridDim.x & 7;
    const uint32_t id = x * (gridDim.x >> 3) + min(x, rem) + (blockIdx.x >> 3);
    const uint32_t band = id / (TR_WINDOW_BAND * (uint32_t)tiles_r), in_band = id - band * (TR_WINDOW_BAND * (uint32_t)tiles_r);
    const uint32_t depth = min((uint32_t)tiles_c - band * TR_WINDOW_BAND, (uint32_t)TR_WINDOW_BAND), tr = in_band / depth;
    const int64_t r0 = (int64_t)tr * TR_WINDOW;
    const int64_t c0 = min((int64_t)(band * TR_WINDOW_BAND + in_band - tr * depth) * 64, cols - 64);

    constexpr int LOADS = IN_ROWS * 8 / NT;
    static_assert(IN_ROWS * 8 % NT == 0 && TR_WINDOW % 64 == 0 && TR_WINDOW * 8 % NT == 0, "whole passes");
    tr_u32x4 v[LOADS];
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
        const int q = t + NT * u;
        const int64_t r = min(max(r0 - 64 + (q >> 3), (int64_t)0), rows - 1);   // a row outside is never stored
        v[u] = *reinterpret_cast<const tr_u32x4_any*>(src + r * cols + c0 + (q & 7) * 8);
    }
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
        const int q = t + NT * u;
#pragma unroll
        for (int d = 0; d < 4; ++d) tile[(q >> 3) * TR_WINDOW_STRIDE + (q & 7) * 4 + d] = v[u][d];
    }
    __syncthreads();
    const uint16_t* const halves = reinterpret_cast<const uint16_t*>(tile);
    const uint32_t phase = (uint32_t)(reinterpret_cast<uintptr_t>(dst) >> 1);
#pragma unroll 2
    for (int u = 0; u < TR_WINDOW * 8 / NT; ++u) {
        const int q = t + NT * u, c = (q >> 3) & 63, p = 64 * (q >> 9) + 8 * (q & 7);   // output row c0 + c, p elements into the window
        const uint32_t shift = (phase + (uint32_t)(c0 + c) * (uint32_t)rows) & 63u;
        const int64_t r = r0 + p - (int)shift;
        const uint16_t* const from = halves + (64 + p - (int)shift) * (2 * TR_WINDOW_STRIDE) + c;
        uint32_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = from[i * (2 * TR_WINDOW_STRIDE)];
        uint16_t* const to = dst + (c0 + c) * rows + r;
        if (r >= 0 && r + 8 <= rows) {
            tr_u32x4 out;
#pragma unroll
            for (int i = 0; i < 4; ++i) out[i] = e[2 * i] | e[2 * i + 1] << 16;
            *reinterpret_cast<tr_u32x4*>(to) = out;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (r + i >= 0 && r + i < rows) to[i] = (uint16_t)e[i];
        }
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
