// The tile kernel for outputs of up to a few hundred tiles: eight waves on one output tile from 64 x 64 to 256 x 128, a ring
// of 64-k stages, one barrier per 64 k.
//
// What bounds such products is the way from the L2 into LDS.  A compute unit receives 150 bytes/ns while every line hits
// in the L2 and 95-125 where a good part of them comes from the memory side (loads alone, 32 KB and more in flight, one
// workgroup on the chip or 256; to LDS or to registers alike); 64 k of a 128 x 128 tile are 32 KB: 0.3 us, where its MFMAs
// take 0.21.  So that path has to be kept busy all the time, with the fewest bytes per flop that leave no unit idle, and
// little else may stand in a row with it:
//
//  * Two waves per SIMD, which cover each other's LDS reads, loads and waits, share one stage and one barrier per 64 k.
//    (The 128 x 128 tile on four waves, one per SIMD, took 0.53-0.56 us per 64 k, slope over K and operands in cache; here 0.31-0.41,
//    and 0.45-0.47 with launch, fill and stores at K = 8192.)
//  * At the barrier every wave has its last fragments of a stage in registers and the loads of the next stage have landed;
//    after it the next stage is read and the released one refilled, NS - 1 iterations ahead of its use.  NS: three stages
//    of the larger tiles are enough (a fourth and fifth gained nothing and lengthen the prologue); 64 x 128 has four (1024 x
//    1600 x 4160 NN 21.5 -> 19.7 us), 64 x 64 five (512 x 512 x 8192 NT 30.6 -> 23.1), two workgroups on a unit.
//  * G = 1: the waves divide the tile and each multiplies both 32-k halves of a stage.  G = 2: two groups of 2 x 2 waves own
//    the whole tile each, group g multiplies half g, and at the end each hands half of its sums to the other through LDS.
//    That costs 0.5 (64 x 64) to 2 us per tile and saves a third of the LDS reads: it is the better form of the 64 x 64 tile
//    (G = 1: 2-7 % slower) and, where an operand is read with the transposing reads, of the 128 x 128 tile over a long K
//    (NN 3-7 %, TN 8-11 % from K = 6000 on; 9-11 % slower below K = 1536); half tiles lose by it.
//  * Tiles of 96 and 192 rows stand between the powers of two, for outputs that those leave a good part of the chip without work of (9 x 18 tiles of
//    128 x 256 are 162 workgroups, 6 x 35 of 192 x 128 are 210).  Not of columns: a wave tile of 48 columns ends rows inside 64 bytes (128 x 96, staged
//    through LDS: NT 1024 x 3072 x 3072 2 % faster than 128 x 128, NN and TN 3 % slower, K = 768 6 %).
//  * Loads are whole 128-byte lines of a K-contiguous operand (a stage row), and whole k-rows of the tile of an
//    MN-contiguous one; both LDS layouts are free of bank conflicts for their reads.
//
// Measured against the kernels that served these products (us, operands in cache, NN / NT / TN):
//   2048 x 4096 x 4096 (256 x 128 tiles) 57 / 54 / 58 -> 51 / 52 / 54;  2048 x 2048 x 8192 (128 x 128) 66 / 66 / 68 -> 58 / 57 / 60;
//   1024 x 1600 x 4160 (64 x 128) 30 / 31 / 30 -> 20 / 20 / 22;  640 x 640 x 2048 (64 x 64) 8.1 / 8.2 / 8.7 -> 6.6 / 6.1 / 7.3;
// and on equal tiles, over 9 000 sampled products, 1.03 (half tiles) to 1.24 times (128 x 128, K >= 3072) as fast as the 32-k
// ring and the four-wave 64-k kernel, none slower by more than 4 %.
//
// MFMA order, accumulator layout and the XCD-aware tile order are those of gemm_tile_kernel16.
#pragma once
#include "gemm_mfma16.hpp"
#include "kernels.hpp"
#include "split_exchange.hpp"

namespace axonn {

// Panels of 96 and 192 rows: some loads are for a part of the wave only.
template <bool PART>
__device__ __forceinline__ void group_load(uint32_t lds_dst, const uint8_t* base, uint32_t voff, uint64_t lanes) {
    if constexpr (PART) direct_load16(lds_dst, base, voff, lanes);
    else direct_load16(lds_dst, base, voff);
}
template <bool PART>
__device__ __forceinline__ void group_load_from(uint32_t lds_dst, const uint8_t* lane_src, uint64_t lanes) {
    if constexpr (PART) direct_load16_from(lds_dst, lane_src, lanes);
    else direct_load16_from(lds_dst, lane_src);
}

// Operand policies: one stage holds ROWS x 64 k of the operand and is filled by all NW waves.
//   issue<X>(stage)           the X-th of this wave's QL direct loads, at the window, into the stage at `stage`
//   issue_tail<X>(...)        the same for a shorter last 64 k
//   advance()                 the window 64 k on
//   cursor<H>(stage, next), read<I>() fragment of 16-row block I: the 32 k of this wave's group (H = 0), or the other half (H = 1)
template <int ROWS, int REGION, int NW, int NB>
struct GroupKContig {   // global P[row * ld + k]; LDS [row][64 k], 16-byte chunks swizzled by (row >> 1) & 7
    static constexpr int BYTES = ROWS * 128;                    // of a stage
    static constexpr int RW = ROWS / NW, QL = (RW + 7) / 8;    // rows per wave; a load is 8 rows x 128 bytes, the last one may be 4
    static_assert(RW * NW == ROWS && RW % 4 == 0, "rows per wave");
    template <int X>
    static constexpr bool half() { return RW - 8 * X == 4; }
    static __device__ __forceinline__ uint32_t row(int x, int lane, int wave) { return RW * wave + 8 * x + (lane >> 3); }
    const uint8_t* base;     // uniform: the wave's first row, at the window
    uint32_t voff[QL];       // per lane
    uint32_t lds_dst;        // uniform
    uint32_t raddr[2];       // read address of block 0 in stage 0, for half 0 (the wave's own) and half 1

    __device__ __forceinline__ void init(const uint16_t* P, int64_t row0, uint32_t ld_bytes, int lane, int wave, int group,
                                         uint32_t lds0, int wave_row) {
        base = reinterpret_cast<const uint8_t*>(P) + (size_t)(row0 + RW * wave) * ld_bytes;
#pragma unroll
        for (int x = 0; x < QL; ++x) {
            voff[x] = (uint32_t)(8 * x + (lane >> 3)) * ld_bytes + ((((uint32_t)lane & 7u) ^ ((row(x, lane, wave) >> 1) & 7u)) << 4);
        }
        lds_dst = lds0 + REGION + (uint32_t)(RW * wave) * 128u;
        const uint32_t r16 = lane & 15, quad = lane >> 4;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            raddr[h] = lds0 + REGION + (uint32_t)(wave_row + r16) * 128u + (((4u * (group ^ h) + quad) ^ (r16 >> 1)) << 4);
    }
    template <int X>
    __device__ __forceinline__ void issue(uint32_t stage) const {
        group_load<half<X>()>(lds_dst + stage + X * 1024u, base, voff[X], 0xFFFFFFFFull);
    }
    template <int X>
    __device__ __forceinline__ void issue_tail(uint32_t stage, size_t delta, int left, int lane, int wave) const {
        const int k = 8 * (int)((lane & 7) ^ ((row(X, lane, wave) >> 1) & 7));
        group_load_from<half<X>()>(lds_dst + stage + X * 1024u, piece_or_zero(base + voff[X] + delta, k < left), 0xFFFFFFFFull);
    }
    __device__ __forceinline__ void advance() { base += 128; }
    struct Cursor {
        uint32_t a;
    };
    template <int H>
    __device__ __forceinline__ Cursor cursor(uint32_t stage, uint32_t) const { return Cursor{raddr[H] + stage}; }
    template <int I>
    __device__ __forceinline__ bf16x8 read(const Cursor& c) const {
        typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<lds_u32x4*>(c.a + I * 2048u));
    }
};

// The same for rows that start anywhere on 16 bytes (a K that is no multiple of 64): every load is still 8 whole lines.  Loaded by k,
// each row's 128 bytes of a stage lie across two lines, each line is fetched for two stages, and a step takes up to 1.6 times as long.
// Here a row that starts s pieces into its line has its last s pieces of every 64 k fetched one stage later, with the rest of
// their line: stage l holds, at the place of piece c, the one of 64 k number l, or, where c + s >= 8, of number l - 1.  An iteration
// reads its own stage and the next one; there is one more stage than iterations, of late pieces only.
template <int ROWS, int REGION, int NW, int NB>
struct GroupKLines {
    using Rows = GroupKContig<ROWS, REGION, NW, NB>;
    static constexpr int BYTES = Rows::BYTES, RW = Rows::RW, QL = Rows::QL;
    template <int X>
    static constexpr bool half() { return Rows::template half<X>(); }
    const uint8_t* base;     // uniform: 128 bytes before the wave's first row, at the window
    uint32_t voff[QL];
    uint32_t lds_dst;
    uint32_t raddr[2];
    uint32_t late[2];        // all ones where this lane reads half 0 (1) from the next stage
    uint32_t late_load;      // bit x: this lane's piece of load x is a late one

    __device__ __forceinline__ void init(const uint16_t* P, int64_t row0, uint32_t ld_bytes, int lane, int wave, int group,
                                         uint32_t lds0, int wave_row) {
        const uint8_t* const first = reinterpret_cast<const uint8_t*>(P) + (size_t)row0 * ld_bytes;
        base = first + (size_t)(RW * wave) * ld_bytes - 128;
        // where a row starts in its line, in pieces: the same for rows 8 apart
        const uint32_t s0 = (uint32_t)(reinterpret_cast<size_t>(first) >> 4), ld = ld_bytes >> 4;
        const uint32_t s = (s0 + Rows::row(0, lane, wave) * ld) & 7u;
        late_load = 0;
#pragma unroll
        for (int x = 0; x < QL; ++x) {
            const uint32_t c = ((uint32_t)lane & 7u) ^ ((Rows::row(x, lane, wave) >> 1) & 7u);
            const bool l = c + s >= 8;
            late_load |= l ? 1u << x : 0u;
            voff[x] = (uint32_t)(8 * x + (lane >> 3)) * ld_bytes + (c << 4) + (l ? 0u : 128u);
        }
        lds_dst = lds0 + REGION + (uint32_t)(RW * wave) * 128u;
        const uint32_t r16 = lane & 15, quad = lane >> 4, s16 = (s0 + r16 * ld) & 7u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t c = 4u * (group ^ h) + quad;
            raddr[h] = lds0 + REGION + (uint32_t)(wave_row + r16) * 128u + ((c ^ (r16 >> 1)) << 4);
            late[h] = c + s16 >= 8 ? ~0u : 0u;
        }
    }
    template <int X>
    __device__ __forceinline__ void issue(uint32_t stage) const {
        group_load<half<X>()>(lds_dst + stage + X * 1024u, base, voff[X], 0xFFFFFFFFull);
    }
    // Stages 0 and 1: the shorter 64 k come first.  `delta`: their bytes behind the row's first k.
    template <int X>
    __device__ __forceinline__ void issue_tail(uint32_t stage, size_t delta, int left, int lane, int wave) const {
        const bool l = late_load >> X & 1;
        group_load_from<half<X>()>(lds_dst + stage + X * 1024u, piece_or_zero(base + voff[X] + delta, !l && tail_k(X, lane, wave) < left), 0xFFFFFFFFull);
    }
    template <int X>
    __device__ __forceinline__ void issue_second(uint32_t stage, size_t delta, int left, int lane, int wave) const {
        const bool l = late_load >> X & 1;
        const uint8_t* const p = base + voff[X];
        group_load_from<half<X>()>(lds_dst + stage + X * 1024u, piece_or_zero(l ? p + 128 + delta : p, !l || tail_k(X, lane, wave) < left), 0xFFFFFFFFull);
    }
    // the stage of late pieces only
    template <int X>
    __device__ __forceinline__ void issue_last(uint32_t stage) const {
        group_load_from<half<X>()>(lds_dst + stage + X * 1024u, piece_or_zero(base + voff[X], late_load >> X & 1), 0xFFFFFFFFull);
    }
    __device__ __forceinline__ void advance() { base += 128; }
    struct Cursor {
        uint32_t a;
    };
    template <int H>
    __device__ __forceinline__ Cursor cursor(uint32_t stage, uint32_t next) const { return Cursor{raddr[H] + stage + (late[H] & (next - stage))}; }
    template <int I>
    __device__ __forceinline__ bf16x8 read(const Cursor& c) const {
        typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<lds_u32x4*>(c.a + I * 2048u));
    }

private:
    __device__ __forceinline__ static int tail_k(int x, int lane, int wave) {
        return 8 * (int)((lane & 7) ^ ((Rows::row(x, lane, wave) >> 1) & 7));
    }
};

template <int ROWS, int REGION, int NW, int NB>
struct GroupMNContig {   // global P[k * ld + row]; LDS [64 k][ROWS], 16-byte chunks swizzled by k
    // a k-row takes up a power of two in LDS; its pieces beyond ROWS are not loaded
    static constexpr int PITCH = ROWS <= 64 ? 64 : ROWS <= 128 ? 128 : 256;
    static constexpr int ROWB = PITCH * 2, CPR = ROWB / 16, BYTES = 64 * ROWB;
    static constexpr bool MASKED = PITCH != ROWS;
    static constexpr int KR = 1024 / ROWB;     // k-rows per load
    static constexpr int QL = 64 / KR / NW;
    static_assert(QL >= 1, "loads per wave");
    const uint8_t* base;     // uniform: the wave's first k-row, at the window
    size_t step_bytes;       // 64 k-rows
    uint32_t voff[QL];
    uint64_t lanes[MASKED ? QL : 1];
    uint32_t lds_dst;
    uint32_t raddr[NB];      // read address of block I in stage 0

    // The transposing read serves its four 16-lane groups (k blocks of eight) two at a time; the eight 32-byte pieces of
    // a pair fall into eight different eighths of the 64 banks.
    static __device__ __forceinline__ uint32_t swizzle(uint32_t k) {
        return PITCH >= 128 ? (2u * (k & 3u)) ^ (8u * ((k >> 3) & 1u)) : (2u * ((k >> 1) & 1u)) ^ (4u * ((k >> 3) & 1u));
    }
    __device__ __forceinline__ void init(const uint16_t* P, int64_t row0, uint32_t ld_bytes, int lane, int wave, int group,
                                         uint32_t lds0, int wave_row) {
        base = reinterpret_cast<const uint8_t*>(P) + (size_t)row0 * 2 + (size_t)(KR * QL * wave) * ld_bytes;
        step_bytes = (size_t)64 * ld_bytes;
        const uint32_t kr = lane / CPR, pos = lane % CPR;
#pragma unroll
        for (int x = 0; x < QL; ++x) {
            const uint32_t piece = pos ^ swizzle(KR * (QL * wave + x) + kr);
            voff[x] = (KR * x + kr) * ld_bytes + (piece << 4);
            if constexpr (MASKED) lanes[x] = __ballot(piece < ROWS / 8);
        }
        lds_dst = lds0 + REGION + (uint32_t)(QL * wave) * 1024u;
        const uint32_t s = lane & 15, k = 32u * group + 8u * (lane >> 4) + (s >> 2);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const uint32_t m = wave_row + 16 * i + 4 * (s & 3);
            raddr[i] = lds0 + REGION + k * ROWB + (((m >> 3) ^ swizzle(k)) << 4) + (m & 4) * 2;
        }
    }
    template <int X>
    __device__ __forceinline__ void issue(uint32_t stage) const {
        group_load<MASKED>(lds_dst + stage + X * 1024u, base, voff[X], lanes[MASKED ? X : 0]);
    }
    template <int X>
    __device__ __forceinline__ void issue_tail(uint32_t stage, size_t delta, int left, int lane, int wave) const {
        const int k = KR * (QL * wave + X) + lane / CPR;
        group_load_from<MASKED>(lds_dst + stage + X * 1024u, piece_or_zero(base + voff[X] + delta, k < left), lanes[MASKED ? X : 0]);
    }
    __device__ __forceinline__ void advance() { base += step_bytes; }
    struct Cursor {
        uint32_t a;
    };
    template <int H>
    __device__ __forceinline__ Cursor cursor(uint32_t stage, uint32_t) const { return Cursor{stage + H * 32u * ROWB}; }
    template <int I>
    __device__ __forceinline__ bf16x8 read(const Cursor& c) const {
        typedef short i16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
        const uint32_t a = raddr[I] + c.a;
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_i16x4*>(a));
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_i16x4*>(a + 4u * ROWB));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
};

// Not the half tiles: LDS has room for three stages of them, one too few for an iteration that reads two (0.83 to 1.02 times as fast).
constexpr bool group_lines(int bm, int bn, bool a_kc, bool b_kc) { return bm + bn <= 256 && (a_kc || b_kc); }
// LINES: an operand is loaded by lines (GroupKLines); an iteration then reads two stages, and one more is there for it where LDS has room
template <int BM, int BN, int G, bool LINES = false, bool A_KC = true, bool B_KC = true>
struct GroupCfg {
    static constexpr int NW = 8, NT = 512;
    static constexpr int WN = G == 2 || BM > BN || BN == 64 ? 2 : 4, WM = NW / G / WN;
    static constexpr int A_BYTES = A_KC ? GroupKContig<BM, 0, NW, 1>::BYTES : GroupMNContig<BM, 0, NW, 1>::BYTES;
    static constexpr int B_BYTES = B_KC ? GroupKContig<BN, 0, NW, 1>::BYTES : GroupMNContig<BN, 0, NW, 1>::BYTES;
    static constexpr int STAGE = A_BYTES + B_BYTES;              // 64 k of both operands
    static constexpr int NS = BM + BN <= 128 ? 5 : BM + BN <= 192 ? 4 + LINES : BM + BN <= 256 ? 3 + LINES : 3;
    static constexpr int EXCHANGE = G == 2 ? BM * BN * 4 : 0;   // half of either group's fp32 tile
    static constexpr int LDS_BYTES = NS * STAGE > EXCHANGE ? NS * STAGE : EXCHANGE;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS per workgroup");
    // 128 registers, so that two workgroups share a compute unit, where LDS has room for two
    static constexpr int WAVES_PER_SIMD = 2 * LDS_BYTES <= 160 * 1024 ? 4 : 2;
};
// of a launch in any layout and form
template <int BM, int BN, int G>
constexpr int group_lds() {
    constexpr bool L = group_lines(BM, BN, true, true);
    constexpr int kc = GroupCfg<BM, BN, G, L>::LDS_BYTES, nn = GroupCfg<BM, BN, G, L, true, false>::LDS_BYTES, tn = GroupCfg<BM, BN, G, false, false, false>::LDS_BYTES;
    return kc > nn ? (kc > tn ? kc : tn) : (nn > tn ? nn : tn);
}

// ---- split-K: the sums of a tile's `splits` workgroups, every one of which adds up and stores a share of the blocks --------------
//
// Range r stores the blocks of its wave tiles that are another's, waits for the others of its tile, and adds up its own: its own
// sum, then the other ranges' in their order (the result does not depend on timing).  All of them move their share at once, where one
// reader per tile takes splits - 1 whole ones while the others' compute units have gone idle.
//
// The workgroups of a tile follow one another in the order of dispatch, and on an idle chip they are there together, or will be as soon as
// the tiles before have ended.  Where they are not (compute units held by other kernels, a stream with a mask of them), a range does not wait for
// long: it hands its share on to one that comes later (split_exchange.hpp), and every workgroup ends whatever else runs.
//
// What it replaces: one reader per tile on the 32-k ring and the four-wave 64-k kernel, half the compute units idle at 120 tiles in two ranges.  us,
// before and here: 1920 x 1024 x 16384 NT 101 -> 70;  640 x 1024 x 8832 NT 37.2 -> 23.2;  256 x 1024 x 12032 NN 30.0 -> 16.5 (six ranges).
// With a counter per tile (a compare-and-swap, a poll and an addition one after the other) the exchange took 8 us longer, with fences 10.
//
// No fences: a device-scope release would write the whole L2 back and an acquire invalidate it, under the other tiles' K loops.  The sums
// leave as device-scope stores that are acknowledged before the flags go out, and come as device-scope loads, past the L2.
struct GroupSplit {
    float* partials;      // [tiles][splits] slots of BM * BN floats: 16 x 16 block, wave, lane
    uint32_t* flags;      // [tiles][splits * (splits - 1)], see split_exchange.hpp
    uint32_t epoch;       // neither 0 nor ~0
    uint32_t probes;      // how often a range looks again for the others before it hands its share on
    int splits;           // 2 .. 6, 8
};

struct GroupSplitWave {
    int lane;
    __device__ __forceinline__ uint32_t load(const uint32_t* p) const { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ void store(uint32_t* p, uint32_t v) const { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ uint32_t exchange(uint32_t* p, uint32_t v) const { return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ bool compare_exchange(uint32_t* p, uint32_t seen, uint32_t v) const {
        return __hip_atomic_compare_exchange_strong(p, &seen, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint64_t ballot(bool b) const { return __ballot(b); }
    __device__ __forceinline__ void pause() const { __builtin_amdgcn_s_sleep(1); }
};
// Device-scope load: from memory, past what this XCD's L2 holds, so that no cache has to be invalidated first.
__device__ __forceinline__ f32x4 load_device_scope(const f32x4* p) {
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    const uint64_t* const q = reinterpret_cast<const uint64_t*>(p);
    const u64x2 v{__hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
    return __builtin_bit_cast(f32x4, v);
}

// The 16 x 16 blocks of a wave tile that are a share.
__device__ __forceinline__ int group_split_first(int share, int blocks, int splits) { return (share * blocks + splits - 1) / splits; }

// device-scope stores and the wait state behind them: see split_k_exchange16
__device__ __forceinline__ void store_device_scope(f32x4* p, const f32x4& v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 0" ::"v"(p), "v"(v) : "memory");
}
// 32 bytes a row: left to the L2 to put together (non-temporal, each went to memory by itself: 640 x 1024 x 8832 NT 23.2 us, 22.6 so)
__device__ __forceinline__ void group_split_store(uint16_t* pc, int ldc, int row_block, int col_block, const f32x4& sum) {
    const u32x2 w{pack2_bf16(sum[0], sum[1]), pack2_bf16(sum[2], sum[3])};
    *reinterpret_cast<u32x2*>(pc + (int64_t)(16 * row_block) * ldc + 16 * col_block) = w;
}

// Returns the shares that are still this workgroup's to settle; its sums of them are in their slots (this wave's, by now).  `pc`, `slots`: this lane's.
template <int MI, int NI, int S, int SLOT>
__device__ __forceinline__ uint32_t group_split_finish(f32x4 (&acc)[MI][NI], const GroupSplit& sp, f32x4* slots, uint32_t* flags, int range, uint16_t* pc, int ldc,
                                                       int wave, int lane, uint32_t* word) {
    constexpr int BLOCKS = MI * NI, NW = 8, OWN = (BLOCKS + S - 1) / S;
    const int first = group_split_first(range, BLOCKS, S), count = group_split_first(range + 1, BLOCKS, S) - first;   // this workgroup's blocks
    f32x4* const mine = slots + (size_t)range * SLOT;
#pragma unroll
    for (int u = 0; u < BLOCKS; ++u)
        if (u < first || u >= first + count) store_device_scope(mine + u * (NW * 64), acc[u / NI][u % NI]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // acknowledged: the compiler does not count stores issued from asm
    __syncthreads();
    if (wave == 0) {
        bool complete;
        const uint32_t held = split_meet(GroupSplitWave{lane}, flags, S, range, sp.epoch, sp.probes, &complete);
        if (lane == 0) *word = held;
    }
    __syncthreads();
    const uint32_t held = __builtin_amdgcn_readfirstlane(*word);
    if (held >> range & 1) {
#pragma unroll
        for (int u = 0; u < BLOCKS; ++u)
            if (u >= first && u < first + count) store_device_scope(mine + u * (NW * 64), acc[u / NI][u % NI]);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return held;
    }
    // all of the other ranges' sums in flight together
    f32x4 v[OWN][S - 1];
#pragma unroll
    for (int i = 0; i < OWN; ++i)
        if (i < count)
#pragma unroll
            for (int q = 0; q < S - 1; ++q)
                v[i][q] = load_device_scope(slots + (size_t)(q + (q >= range ? 1 : 0)) * SLOT + (first + i) * (NW * 64));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < OWN; ++i)
        if (i < count) {
            f32x4 sum;
#pragma unroll
            for (int u = 0; u < BLOCKS; ++u)
                if (u == first + i) sum = acc[u / NI][u % NI];
#pragma unroll
            for (int q = 0; q < S - 1; ++q) sum += v[i][q];
            group_split_store(pc, ldc, (first + i) / NI, (first + i) % NI, sum);
        }
    return held;
}
// The shares that were handed on: rare, and off the path above.  The sums are added in the same order, the share's own range's first.
template <int MI, int NI, int SLOT>
__device__ __forceinline__ void group_split_settle(uint32_t held, const GroupSplit& sp, const f32x4* slots, uint32_t* flags, uint16_t* pc, int ldc, int wave, int lane, uint32_t* word) {
    constexpr int BLOCKS = MI * NI, NW = 8;
    while (held) {
        const int share = __builtin_ctz(held);
        held &= held - 1;
        __syncthreads();   // every wave's sums are in memory, and every wave has read the word
        if (wave == 0) {
            const bool all = split_settle(GroupSplitWave{lane}, flags, sp.splits, share, sp.epoch);
            if (lane == 0) *word = all;
        }
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(*word)) continue;
        const int end = group_split_first(share + 1, BLOCKS, sp.splits);
        for (int u = group_split_first(share, BLOCKS, sp.splits); u < end; ++u) {
            const f32x4* const p = slots + u * (NW * 64);
            f32x4 sum = load_device_scope(p + (size_t)share * SLOT);
            for (int q = 0; q < sp.splits; ++q)
                if (q != share) sum += load_device_scope(p + (size_t)q * SLOT);
            group_split_store(pc, ldc, u / NI, u % NI, sum);
        }
    }
}

// One tile.  LINES: its K-contiguous operands by lines; K > 64 NS.  SPLITK: one of the K ranges of a tile.
template <int BM, int BN, int G, bool A_KC, bool B_KC, bool KTAIL, bool LINES, bool SPLITK = false>
__device__ __forceinline__ void group_tile(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, uint16_t* __restrict__ C,
                                           int K, int lda, int ldb, int ldc, int64_t m0, int64_t n0, int k_tail,
                                           const GroupSplit& split = GroupSplit{}, int tile = 0, int range = 0) {
    constexpr bool LINES_A = LINES && A_KC, LINES_B = LINES && B_KC;
    using Cfg = GroupCfg<BM, BN, G, LINES, A_KC, B_KC>;
    constexpr int NW = Cfg::NW, NS = Cfg::NS;
    constexpr int AHEAD = LINES ? 2 : 1;   // an iteration reads this many stages
    constexpr uint32_t STAGE = Cfg::STAGE;
    constexpr int TM = BM / Cfg::WM, TN = BN / Cfg::WN, MI = TM / 16, NI = TN / 16, NM = MI * NI;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const int t = threadIdx.x;
    int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int group = G == 2 ? wave >> 2 : 0, wm = (G == 2 ? wave & 3 : wave) / Cfg::WN, wn = wave % Cfg::WN;

    using OpA = typename std::conditional<LINES_A, GroupKLines<BM, 0, NW, MI>,
                                          typename std::conditional<A_KC, GroupKContig<BM, 0, NW, MI>, GroupMNContig<BM, 0, NW, MI>>::type>::type;
    using OpB = typename std::conditional<LINES_B, GroupKLines<BN, Cfg::A_BYTES, NW, NI>,
                                          typename std::conditional<B_KC, GroupKContig<BN, Cfg::A_BYTES, NW, NI>, GroupMNContig<BN, Cfg::A_BYTES, NW, NI>>::type>::type;
    constexpr int QLA = OpA::QL, QLB = OpB::QL, QL = QLA + QLB;
    constexpr int QX = (LINES_A ? QLA : 0) + (LINES_B ? QLB : 0);   // loads of the stage of late pieces
    const uint32_t lds0 = lds_address(smem);
    OpA opa;
    OpB opb;
    opa.init(A, m0, 2u * (uint32_t)lda, lane, wave, group, lds0, wm * TM);
    opb.init(B, n0, 2u * (uint32_t)ldb, lane, wave, group, lds0, wn * TN);

    f32x4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    struct Frags {
        bf16x8 a[MI], b[NI];
    };
    Frags f[2];

#define AXONN_FENCE() __builtin_amdgcn_sched_barrier(0)
    auto issue_stage = [&](uint32_t stage) __attribute__((always_inline)) {
        static_for<QLA>([&](auto x) __attribute__((always_inline)) { opa.template issue<decltype(x)::value>(stage); });
        static_for<QLB>([&](auto x) __attribute__((always_inline)) { opb.template issue<decltype(x)::value>(stage); });
        opa.advance();
        opb.advance();
    };
    auto issue_last = [&](auto x_c, uint32_t stage) __attribute__((always_inline)) {
        constexpr int X = decltype(x_c)::value;
        if constexpr (X < QLA) {
            if constexpr (LINES_A) opa.template issue_last<X>(stage);
        } else {
            if constexpr (LINES_B) opb.template issue_last<X - QLA>(stage);
        }
    };
    // fragments of the iteration whose stage is `stage`; `after`: the stage behind it
    auto read_range = [&](Frags& x, uint32_t stage, uint32_t after, auto h_c, auto lo_c, auto hi_c) __attribute__((always_inline)) {
        constexpr int LO = decltype(lo_c)::value, HI = decltype(hi_c)::value;
        constexpr int H = decltype(h_c)::value;
        const auto ca = opa.template cursor<H>(stage, after);
        const auto cb = opb.template cursor<H>(stage, after);
        static_for<HI - LO>([&](auto d) __attribute__((always_inline)) {
            constexpr int X = LO + decltype(d)::value;
            if constexpr (X < MI)
                x.a[X] = opa.template read<X>(ca);
            else
                x.b[X - MI] = opb.template read<X - MI>(cb);
        });
    };
    auto mfma_range = [&](const Frags& x, auto lo_c, auto hi_c) __attribute__((always_inline)) {
        constexpr int LO = decltype(lo_c)::value, HI = decltype(hi_c)::value;
        static_for<HI - LO>([&](auto d) __attribute__((always_inline)) {
            constexpr int I = (LO + decltype(d)::value) / NI, J0 = (LO + decltype(d)::value) % NI;
            constexpr int J = (I & 1) ? NI - 1 - J0 : J0;
            acc[I][J] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.b[J], x.a[I], acc[I][J], 0, 0, 0);
        });
    };

    // ---- prologue: the first stages
    const int KI = K / 64;
    const int fill = LINES || KI > NS ? NS : KI;
    {
        int s = 0;
        if constexpr (KTAIL) {
            const size_t whole = (size_t)(K - 64);
            static_for<QLA>([&](auto x) __attribute__((always_inline)) {
                opa.template issue_tail<decltype(x)::value>(0u, 2 * (A_KC ? whole : whole * lda), k_tail, lane, wave);
            });
            static_for<QLB>([&](auto x) __attribute__((always_inline)) {
                opb.template issue_tail<decltype(x)::value>(0u, 2 * (B_KC ? whole : whole * ldb), k_tail, lane, wave);
            });
            s = 1;
            if constexpr (LINES) {
                static_for<QLA>([&](auto x) __attribute__((always_inline)) {
                    if constexpr (LINES_A) opa.template issue_second<decltype(x)::value>(STAGE, 2 * whole, k_tail, lane, wave);
                    else opa.template issue<decltype(x)::value>(STAGE);
                });
                static_for<QLB>([&](auto x) __attribute__((always_inline)) {
                    if constexpr (LINES_B) opb.template issue_second<decltype(x)::value>(STAGE, 2 * whole, k_tail, lane, wave);
                    else opb.template issue<decltype(x)::value>(STAGE);
                });
                opa.advance();
                opb.advance();
                s = 2;
            }
        }
        for (; s < fill; ++s) issue_stage(s * STAGE);
    }
    if (!LINES && KI < NS) {   // all of K is in LDS
        asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        for (int i = 0; i < KI; ++i) {
            static_for<2 / G>([&](auto h) __attribute__((always_inline)) {
                read_range(f[0], i * STAGE, (i + 1) * STAGE, h, Int<0>{}, Int<MI + NI>{});
                mfma_range(f[0], Int<0>{}, Int<NM>{});
            });
        }
    } else {
        constexpr int P = NM < 4 ? 0 : 2;   // MFMAs before the barrier
        // clusters of reads and loads: no difference in time, but other numbers make the compiler spill
        constexpr int NC = BM * BN <= 64 * 128 ? 3 : 2;
        uint32_t st = 0;                // stage of the running iteration
        auto next = [&](uint32_t s) __attribute__((always_inline)) { return s + STAGE == NS * STAGE ? 0u : s + STAGE; };
        // MFMAs on `cur`, among them the reads of `nxt` from half H of stage `from` and the loads LF .. LL-1 of a stage
        // into `to` (LATE: of the stage of late pieces).  VM >= 0: a barrier first, at which this wave's fragments are in registers
        // and all its loads but the last VM have landed.
        auto substep = [&](const Frags& cur, Frags& nxt, auto vm_c, auto read_c, auto h_c, auto lf_c, auto ll_c, auto late_c, uint32_t from, uint32_t to) __attribute__((always_inline)) {
            constexpr bool READ = decltype(read_c)::value, LATE = decltype(late_c)::value;
            const uint32_t after = next(from);
            constexpr int VM = decltype(vm_c)::value, LF = decltype(lf_c)::value, NL = decltype(ll_c)::value - LF;
            AXONN_FENCE();
            mfma_range(cur, Int<0>{}, Int<P>{});
            AXONN_FENCE();
            if constexpr (VM >= 0) {
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(VM < 0 ? 0 : VM) : "memory");
                AXONN_FENCE();
            }
            constexpr int R = NM - P;
            static_for<NC>([&](auto q_c) __attribute__((always_inline)) {
                constexpr int Q = decltype(q_c)::value;
                if constexpr (READ) read_range(nxt, from, after, h_c, Int<Q * (MI + NI) / NC>{}, Int<(Q + 1) * (MI + NI) / NC>{});
                static_for<(Q + 1) * NL / NC - Q * NL / NC>([&](auto d) __attribute__((always_inline)) {
                    constexpr int X = LF + Q * NL / NC + decltype(d)::value;
                    if constexpr (LATE)
                        issue_last(Int<X>{}, to);
                    else if constexpr (X < QLA)
                        opa.template issue<X>(to);
                    else
                        opb.template issue<X - QLA>(to);
                });
                AXONN_FENCE();
                __builtin_amdgcn_s_setprio(1);
                mfma_range(cur, Int<P + Q * R / NC>{}, Int<P + (Q + 1) * R / NC>{});
                __builtin_amdgcn_s_setprio(0);
                AXONN_FENCE();
            });
        };
        using Yes = std::true_type;
        using No = std::false_type;
        wait_vmcnt<(NS - AHEAD) * QL>();
        __builtin_amdgcn_s_barrier();
        AXONN_FENCE();
        // what may be in flight at the barrier of an iteration: the stages beyond those that the next one reads
        constexpr int VM = (NS - 1 - AHEAD) * QL;
        // at the J-th of the last NS ones; < 0: no barrier
        constexpr auto vm_at_end = [](int j) {
            const int stages = NS - 1 - AHEAD - j;   // whole ones
            return j == NS - 1 ? -1 : (stages > 0 ? stages * QL : 0) + (LINES && j > 0 && stages >= 0 ? QX : 0);
        };
        if constexpr (G == 2) {
            // one iteration: multiplies `cur`, reads the next iteration's fragments, refills the stage behind the barrier
            auto step = [&](const Frags& cur, Frags& nxt, auto vm_c, auto read_c, auto load_c, auto late_c) __attribute__((always_inline)) {
                const uint32_t ns = next(st);
                substep(cur, nxt, vm_c, read_c, Int<0>{}, Int<0>{}, Int<decltype(load_c)::value || decltype(late_c)::value ? QL : 0>{}, late_c, ns, st);
                if constexpr (decltype(load_c)::value) {
                    opa.advance();
                    opb.advance();
                }
                st = ns;
            };
            int n = KI - NS;   // iterations with a load; the register buffers alternate, and the ones without a load start on f[0]
            if (n & 1) {
                read_range(f[1], 0u, STAGE, Int<0>{}, Int<0>{}, Int<MI + NI>{});
                step(f[1], f[0], Int<VM>{}, Yes{}, Yes{}, No{});
            } else {
                read_range(f[0], 0u, STAGE, Int<0>{}, Int<0>{}, Int<MI + NI>{});
            }
            for (n >>= 1; n > 0; --n) {
                step(f[0], f[1], Int<VM>{}, Yes{}, Yes{}, No{});
                step(f[1], f[0], Int<VM>{}, Yes{}, Yes{}, No{});
            }
            static_for<NS>([&](auto j_c) __attribute__((always_inline)) {
                constexpr int J = decltype(j_c)::value;
                step(f[J & 1], f[1 - (J & 1)], Int<vm_at_end(J)>{}, std::bool_constant<(J < NS - 1)>{}, No{}, std::bool_constant<(LINES && J == 0)>{});
            });
        } else {
            // one iteration: both halves.  The stage is released at the barrier in the second one; its loads go out there
            // and in the next iteration's first half.
            constexpr int QH = QL / 2;
            uint32_t to = 0;
            // loads of the first and of the second substep: 0 none, 1 a stage's, 2 those of the stage of late pieces
            auto step = [&](auto vm_c, auto last_c, auto load0_c, auto load1_c) __attribute__((always_inline)) {
                constexpr bool LAST = decltype(last_c)::value;
                constexpr int L0 = decltype(load0_c)::value, L1 = decltype(load1_c)::value;
                const uint32_t ns = next(st);
                substep(f[0], f[1], Int<-1>{}, Yes{}, Int<1>{}, Int<QH>{}, Int<L0 ? QL : QH>{}, std::bool_constant<L0 == 2>{}, st, to);
                if constexpr (L0 == 1) {
                    opa.advance();
                    opb.advance();
                }
                substep(f[1], f[0], vm_c, std::bool_constant<!LAST>{}, Int<0>{}, Int<0>{}, Int<L1 ? QH : 0>{}, std::bool_constant<L1 == 2>{}, ns, st);
                to = st;
                st = ns;
            };
            read_range(f[0], 0u, STAGE, Int<0>{}, Int<0>{}, Int<MI + NI>{});
            int n = KI - NS;
            using L0 = Int<0>;
            using L1 = Int<1>;
            using L2 = Int<LINES ? 2 : 0>;
            if (n > 0) {
                step(Int<VM>{}, No{}, L0{}, L1{});
                for (; n > 1; --n) step(Int<VM>{}, No{}, L1{}, L1{});
                step(Int<VM>{}, No{}, L1{}, L2{});
            } else {
                step(Int<VM>{}, No{}, L0{}, L2{});
            }
            static_for<NS - 1>([&](auto j_c) __attribute__((always_inline)) {
                constexpr int J = decltype(j_c)::value + 1;
                step(Int<vm_at_end(J)>{}, std::bool_constant<(J == NS - 1)>{}, Int<LINES && J == 1 ? 2 : 0>{}, L0{});
            });
        }
    }
    if constexpr (!SPLITK) __syncthreads();   // the stages are free
    asm volatile("" : "+v"(lane));   // see split_k_exchange16: keeps the epilogue's addresses out of the K loop's registers
    if constexpr (SPLITK) {
        static_assert(G == 1, "the waves divide the tile");
        uint16_t* const pc = C + (m0 + wm * TM) * (int64_t)ldc + n0 + wn * TN;
        constexpr int SLOT = BM * BN / 4;   // f32x4 of a slot
        f32x4* const slots = reinterpret_cast<f32x4*>(split.partials) + (size_t)tile * split.splits * SLOT + wave * 64 + lane;
        uint32_t* const flags = split.flags + tile * split.splits * (split.splits - 1);
        uint16_t* const mine = pc + (int64_t)(lane & 15) * ldc + 4 * (lane >> 4);
        uint32_t* const word = reinterpret_cast<uint32_t*>(smem);   // behind the barriers of the exchange the stages are free
        uint32_t held = 0;
        switch (split.splits) {
            case 2: held = group_split_finish<MI, NI, 2, SLOT>(acc, split, slots, flags, range, mine, ldc, wave, lane, word); break;
            case 3: held = group_split_finish<MI, NI, 3, SLOT>(acc, split, slots, flags, range, mine, ldc, wave, lane, word); break;
            case 4: held = group_split_finish<MI, NI, 4, SLOT>(acc, split, slots, flags, range, mine, ldc, wave, lane, word); break;
            case 5: held = group_split_finish<MI, NI, 5, SLOT>(acc, split, slots, flags, range, mine, ldc, wave, lane, word); break;
            case 6: held = group_split_finish<MI, NI, 6, SLOT>(acc, split, slots, flags, range, mine, ldc, wave, lane, word); break;
            default: held = group_split_finish<MI, NI, 8, SLOT>(acc, split, slots, flags, range, mine, ldc, wave, lane, word); break;
        }
        if (__builtin_expect(held != 0, 0)) group_split_settle<MI, NI, SLOT>(held, split, slots, flags, mine, ldc, wave, lane, word);
    } else if constexpr (G == 1) {
        uint8_t* const epi = smem + wave * (32 * TN);
        uint16_t* const pc = C + (m0 + wm * TM) * (int64_t)ldc + n0 + wn * TN;
#pragma unroll
        for (int i = 0; i < MI; ++i) store_block_row16<TN, NI>(acc[i], epi, pc + (int64_t)(16 * i) * ldc, ldc, lane);
    } else {
        // the groups' sums: group 0 keeps the first half of the block rows, group 1 the second
        constexpr int MH = MI / 2;
        f32x4* const slots = reinterpret_cast<f32x4*>(smem);
        f32x4* const mine = slots + wave * (MH * NI * 64) + lane;
        const f32x4* const other = slots + (wave ^ 4) * (MH * NI * 64) + lane;
        f32x4 out[MH][NI];
        auto give = [&](auto first_c) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < MH; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) mine[(i * NI + j) * 64] = acc[decltype(first_c)::value + i][j];
        };
        auto take = [&](auto first_c) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < MH; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) out[i][j] = acc[decltype(first_c)::value + i][j] + other[(i * NI + j) * 64];
        };
        if (group == 0) give(Int<MH>{});
        else give(Int<0>{});
        __syncthreads();
        if (group == 0) take(Int<0>{});
        else take(Int<MH>{});
        // staged through the slot that this wave alone has read
        uint8_t* const epi = smem + (wave ^ 4) * (MH * NI * 1024);
        uint16_t* const pc = C + (m0 + wm * TM + group * (TM / 2)) * (int64_t)ldc + n0 + wn * TN;
#pragma unroll
        for (int i = 0; i < MH; ++i) store_block_row16<TN, NI>(out[i], epi, pc + (int64_t)(16 * i) * ldc, ldc, lane);
    }
#undef AXONN_FENCE
}

// The same over `split.splits` K ranges per tile, of K / 64 / splits or one more 64 k; whole tiles, K >= 64 splits.
template <int BM, int BN, bool A_KC, bool B_KC>
__global__ __launch_bounds__(512, (GroupCfg<BM, BN, 1>::WAVES_PER_SIMD)) void gemm_tile_kernel_k64gs(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, uint16_t* __restrict__ C,
    int K, int lda, int ldb, int ldc, int tiles_m, int tiles_n, int group_m, GroupSplit split) {
    const int tiles = tiles_m * tiles_n, nwg = tiles * split.splits;
    // XCD x runs the workgroups x, x + 8, ...: a contiguous chunk of the sequence (tile, range), see map_workgroup
    const int x = blockIdx.x & 7, rem = nwg & 7;
    const int id = x * (nwg >> 3) + (x < rem ? x : rem) + (blockIdx.x >> 3);
    const int tile = id / split.splits, range = id - tile * split.splits;
    const int group_sz = group_m * tiles_n, group = tile / group_sz, first_m = group * group_m;
    const int gm = min(tiles_m - first_m, group_m), in_group = tile - group * group_sz;
    const int64_t m0 = (int64_t)(first_m + in_group % gm) * BM, n0 = (int64_t)(in_group / gm) * BN;
    const int steps = K / 64, each = steps / split.splits, more = steps - each * split.splits;
    const int64_t k0 = 64 * (int64_t)(each * range + min(range, more));
    group_tile<BM, BN, 1, A_KC, B_KC, false, false, true>(A + (A_KC ? k0 : k0 * lda), B + (B_KC ? k0 : k0 * ldb), C,
                                                         64 * (each + (range < more ? 1 : 0)), lda, ldb, ldc, m0, n0, 0, split, tile, range);
}

// Requires M >= BM, N >= BN, K % 64 == 0 (KTAIL: see TileGrid), and 16-byte aligned rows.
template <int BM, int BN, int G, bool A_KC, bool B_KC, bool KTAIL = false>
__global__ __launch_bounds__(512, (GroupCfg<BM, BN, G>::WAVES_PER_SIMD)) void gemm_tile_kernel_k64g(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, uint16_t* __restrict__ C,
    int K, int lda, int ldb, int ldc, TileGrid grid, int group_m, SplitK sk) {
    const TileWork work = map_workgroup<false, false>(blockIdx.x, grid.tiles_m * grid.tiles_n, K, grid.tiles_m, grid.tiles_n, group_m, sk);
    const int64_t m0 = min(work.tile_m * BM, grid.m_last), n0 = min(work.tile_n * BN, grid.n_last);
    if constexpr (KTAIL && group_lines(BM, BN, A_KC, B_KC)) {
        if (__builtin_expect(K <= kGroupLinesK, 1))
            group_tile<BM, BN, G, A_KC, B_KC, true, false>(A, B, C, K, lda, ldb, ldc, m0, n0, grid.k_tail);
        else
            group_tile<BM, BN, G, A_KC, B_KC, true, true>(A, B, C, K, lda, ldb, ldc, m0, n0, grid.k_tail);
    } else {
        group_tile<BM, BN, G, A_KC, B_KC, KTAIL, false>(A, B, C, K, lda, ldb, ldc, m0, n0, grid.k_tail);
    }
}

}  // namespace axonn
