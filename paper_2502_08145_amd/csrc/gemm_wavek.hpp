// The wave-K kernel: the product
//
//   C[M,N] = sum_k a(i,k) b(k,j)      (the local matrix multiply of Algorithm 1 lines 3, 11, 13)
//
// for outputs of few tiles, for few rows, and for operands whose rows start at any 2-byte address.
//
// Such products are bound by latency: a tile kernel gives every output tile ONE workgroup that walks all
// of K through barriers, so a small output leaves most compute units idle behind a serial chain.  Here
// the chain is cut inside the workgroup: its waves all own the SAME output tile (16 MI x 16 NI), and wave w
// takes the 64-k chunks w, w + WK, w + 2 WK, ... of the reduction.  A wave shares nothing with the others
// until the end, so there is no barrier in the loop, and the loads of a chunk per wave are in flight all the
// time.  At the end the partial accumulators go through LDS once and are added in the order of
// the waves (the result does not depend on timing).  No scratch memory is needed.
//
//  * Either kind of operand goes through a region of LDS that belongs to the wave alone.  A wave's LDS operations
//    execute in order, so its region needs no barrier.
//  * A K-contiguous operand (A of NN/NT, B of NT) is loaded 8 rows x 128 bytes, whole lines, at a time, kept as
//    [16 MI][64 k], padded by 16 bytes a row, and read with ds_read_b128.  (Loaded straight into the registers of the
//    MFMA operand, sixteen half lines at a time, 24 x 2048 x 8192 NT took 18 us where this takes 11.)
//  * An MN-contiguous operand (A of TN, B of NN/TN) is kept as in memory, [64 k][16 NI], padded likewise, and read
//    with the transposing ds_read_b64_tr_b16.
//  * Loads are 16 bytes at 2-byte alignment: the hardware takes them at any address, a little slower where
//    a line is crossed (fetched element by element, as a guarded kernel would, the same product is ten times
//    slower).  Nothing outside the operands is read: the last tile of a row or column of tiles is moved
//    back so that it ends at the matrix' edge (it then computes some outputs a second time, to the same
//    bits); rows of a K-contiguous operand with fewer rows than a tile are clamped; the pieces of the last
//    chunk that lie across K are fetched K-aligned from the end and shifted, those beyond K are zero.
//
// Requires leading dimensions below 2^24; K >= 8 if an operand is K-contiguous; M >= 16 MI if A is MN-contiguous
// or MI > 2, N >= 16 NI if B is or NI > 2.
#pragma once
#include "gemm_mfma.hpp"
#include "gemm_mfma16.hpp"

namespace axonn {

struct WaveKCfg {
    static constexpr int KC = 64;            // k per chunk
    static constexpr int64_t MAX_LD = (int64_t)1 << 24;
    // two waves per SIMD with 256 registers each, four with 128 where the tile is small enough
    static constexpr int max_waves(int mi, int ni) { return mi * ni <= 2 ? 16 : 8; }
    static constexpr int PAD = 16;           // bytes behind every row in LDS
    static constexpr int stage_bytes(bool kc, int blocks) { return kc ? 16 * blocks * (2 * KC + PAD) : KC * (32 * blocks + PAD); }
    static constexpr int lds_bytes(bool a_kc, bool b_kc, int mi, int ni, int wk) {
        const int st = wk * (stage_bytes(a_kc, mi) + stage_bytes(b_kc, ni)), red = wk > 1 ? wk * mi * ni * 1024 : 0;
        return st > red ? st : red;
    }
};

// 128 bits moved right by `s` 16-bit elements (s >= 8: nothing is left)
__device__ __forceinline__ u32x4 shift_out_elements(u32x4 v, int s) {
    if (s >= 8) return u32x4{0u, 0u, 0u, 0u};
    unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v);
    x >>= 16 * s;
    return __builtin_bit_cast(u32x4, x);
}

// Addresses are a wave-uniform 64-bit base that moves along k and 32-bit per-lane byte offsets, which hold
// at most 64 rows of a K-contiguous operand or 32 k-rows of an MN-contiguous one: ld < 2^24.
//
// A wave's share of one K-contiguous operand: 16 NB rows.
template <int NB>
struct WaveKContig {
    static constexpr int ROWB = 2 * WaveKCfg::KC + WaveKCfg::PAD;   // bytes per row in LDS
    static constexpr int LDS_BYTES = 16 * NB * ROWB;
    static constexpr int NL = 2 * NB;                               // loads per chunk, 8 rows x 128 bytes each
    // Only tiles of one and two blocks may have fewer rows than the tile: they hold the (clamped) row of
    // every load in a register; the larger ones step from load to load in the scalar base.
    static constexpr bool CLAMP = NB <= 2;
    const uint8_t* base;       // uniform: row 0 of the tile, k = 0
    int64_t ld_bytes;
    uint32_t piece[CLAMP ? NL : 1];   // this lane's piece of load j: row 8 j + lane/8, k = 8 (lane % 8)
    uint32_t wr, rd;           // LDS byte offsets: where this lane's piece goes; where it reads block 0
    struct Regs {
        u32x4 v[NL];
    };
    __device__ __forceinline__ void init(const uint16_t* P, int64_t row0, int64_t rows, int64_t ld, int lane) {
        base = reinterpret_cast<const uint8_t*>(P + row0 * ld);
        ld_bytes = 2 * ld;
        const int last = (int)(rows - row0 < 16 * NB ? rows - row0 : 16 * NB) - 1;
#pragma unroll
        for (int j = 0; j < (CLAMP ? NL : 1); ++j) {
            int r = 8 * j + (lane >> 3);
            r = r < last ? r : last;   // fewer rows than a tile: the last one again (never stored)
            piece[j] = (uint32_t)r * (uint32_t)ld_bytes + 16u * (lane & 7);
        }
        wr = (uint32_t)((lane >> 3) * ROWB + 16 * (lane & 7));
        rd = (uint32_t)((lane & 15) * ROWB + 16 * (lane >> 4));
    }
    __device__ __forceinline__ u32x4 fetch(const uint8_t* p, int j) const {
        if constexpr (CLAMP)
            return *reinterpret_cast<const u32x4_any*>(p + piece[j]);
        else
            return *reinterpret_cast<const u32x4_any*>(p + 8 * j * ld_bytes + piece[0]);
    }
    __device__ __forceinline__ void load(Regs& x, int64_t k0) const {
        const uint8_t* const p = base + 2 * k0;
#pragma unroll
        for (int j = 0; j < NL; ++j) x.v[j] = fetch(p, j);
    }
    // the last, shorter chunk, of which `left` (1 .. 63) k exist
    __device__ __forceinline__ void load_tail(Regs& x, int64_t k0, int left, int lane) const {
        const int kq = 8 * (lane & 7), s = kq > left - 8 ? kq - (left - 8) : 0;   // a piece across K or beyond: s elements back
        const uint8_t* const p = base + 2 * k0;
#pragma unroll
        for (int j = 0; j < NL; ++j) x.v[j] = shift_out_elements(fetch(p - 2 * s, j), s);
    }
    __device__ __forceinline__ void stage(const Regs& x, uint8_t* lds) const {
#pragma unroll
        for (int j = 0; j < NL; ++j) *reinterpret_cast<u32x4*>(lds + wr + j * (8 * ROWB)) = x.v[j];
    }
    __device__ __forceinline__ bf16x8 fragment(const uint8_t* lds, int b, int h) const {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(lds + rd + b * (16 * ROWB) + h * 64));
    }
};

// A wave's share of one MN-contiguous operand: 16 NB rows (m or n) of it.
template <int NB>
struct WaveMNContig {
    static constexpr int ROWB = 32 * NB + WaveKCfg::PAD;   // bytes per k-row in LDS
    static constexpr int LDS_BYTES = WaveKCfg::KC * ROWB;
    static constexpr int PPR = 2 * NB;                        // 16-byte pieces per k-row
    static constexpr int KR = 64 / PPR;                       // k-rows per load
    static constexpr int NL = WaveKCfg::KC / KR;              // loads per chunk
    const uint8_t* base;       // uniform: k-row 0, first row (m or n) of the tile
    int64_t ld_bytes;
    uint32_t piece;            // this lane's piece of k-row (lane / PPR)
    int kr;
    uint32_t wr, rd;           // LDS byte offsets: where this lane's piece goes; where it reads block 0
    struct Regs {
        u32x4 v[NL];
    };
    __device__ __forceinline__ void init(const uint16_t* P, int64_t row0, int64_t /*rows*/, int64_t ld, int lane) {
        base = reinterpret_cast<const uint8_t*>(P + row0);
        ld_bytes = 2 * ld;
        kr = lane / PPR;
        piece = (uint32_t)kr * (uint32_t)ld_bytes + 16u * (lane % PPR);
        wr = (uint32_t)(kr * ROWB + 16 * (lane % PPR));
        // the 16 lanes of group g = lane/16 address k-rows 8g .. 8g+3 (then + 4), four rows of the block each
        const int s = lane & 15, g = lane >> 4;
        rd = (uint32_t)((8 * g + (s >> 2)) * ROWB + 8 * (s & 3));
    }
    __device__ __forceinline__ void load(Regs& x, int64_t k0) const {
        const uint8_t* p = base + k0 * ld_bytes;
#pragma unroll
        for (int j = 0; j < NL; ++j, p += KR * ld_bytes) x.v[j] = *reinterpret_cast<const u32x4_any*>(p + piece);
    }
    __device__ __forceinline__ void load_tail(Regs& x, int64_t k0, int left, int /*lane*/) const {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            x.v[j] = u32x4{0u, 0u, 0u, 0u};
            if (j * KR < left) {   // uniform
                // k-rows behind K: the lane takes its piece from the last one that exists, and drops it
                const int over = j * KR + kr - (left - 1);
                const uint32_t back = over > 0 ? (uint32_t)over * (uint32_t)ld_bytes : 0u;
                const u32x4 v = *reinterpret_cast<const u32x4_any*>(base + (k0 + j * KR) * ld_bytes + (piece - back));
                if (over <= 0) x.v[j] = v;
            }
        }
    }
    __device__ __forceinline__ void stage(const Regs& x, uint8_t* lds) const {
#pragma unroll
        for (int j = 0; j < NL; ++j) *reinterpret_cast<u32x4*>(lds + wr + j * (KR * ROWB)) = x.v[j];
    }
    __device__ __forceinline__ bf16x8 fragment(const uint8_t* lds, int b, int h) const {
        typedef short i16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
        const uint8_t* p = lds + rd + h * (32 * ROWB) + 32 * b;
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p));
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + 4 * ROWB));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
};

// LDS accesses of this wave before and after stay in order (the hardware keeps them so; the compiler must too)
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// blockDim.x = 64 * (waves per tile); dynamic LDS: WaveKCfg::lds_bytes.
template <bool A_KC, bool B_KC, int MI, int NI>
__global__ __launch_bounds__(64 * WaveKCfg::max_waves(MI, NI)) void gemm_wavek_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, uint16_t* __restrict__ C, int64_t M, int64_t N, int64_t K,
    int64_t lda, int64_t ldb, int64_t ldc, int tiles_m, int tiles_n, int group_m) {
    constexpr int TM = 16 * MI, TN = 16 * NI;
    using OpA = typename std::conditional<A_KC, WaveKContig<MI>, WaveMNContig<MI>>::type;
    using OpB = typename std::conditional<B_KC, WaveKContig<NI>, WaveMNContig<NI>>::type;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), waves = blockDim.x >> 6;

    const TileWork work = map_workgroup<false, false>(blockIdx.x, gridDim.x, 0, tiles_m, tiles_n, group_m, SplitK{});
    int64_t m0 = (int64_t)work.tile_m * TM, n0 = (int64_t)work.tile_n * TN;
    m0 = m0 + TM <= M ? m0 : M > TM ? M - TM : 0;
    n0 = n0 + TN <= N ? n0 : N > TN ? N - TN : 0;

    OpA opa;
    OpB opb;
    opa.init(A, m0, M, lda, lane);
    opb.init(B, n0, N, ldb, lane);
    uint8_t* const la = smem + wave * (OpA::LDS_BYTES + OpB::LDS_BYTES);
    uint8_t* const lb = la + OpA::LDS_BYTES;

    f32x4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    struct Regs {
        typename OpA::Regs a;
        typename OpB::Regs b;
    };
    Regs r;
    auto load = [&](int64_t k0) __attribute__((always_inline)) {
        opa.load(r.a, k0);
        opb.load(r.b, k0);
    };
    auto stage = [&]() __attribute__((always_inline)) {
        opa.stage(r.a, la);
        opb.stage(r.b, lb);
        wave_order();
    };
    auto multiply_half = [&](int h) __attribute__((always_inline)) {
        bf16x8 fa[MI], fb[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) fa[i] = opa.fragment(la, i, h);
#pragma unroll
        for (int j = 0; j < NI; ++j) fb[j] = opb.fragment(lb, j, h);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    };
    // whole chunks: wave, wave + waves, ...; a shorter one at the end is the first of the wave that has the
    // fewest (its loads need the extra code in one place only then)
    const int64_t step = (int64_t)waves * WaveKCfg::KC, Kw = K & ~(int64_t)(WaveKCfg::KC - 1);
    const int left = (int)(K - Kw);
    const bool tail = left != 0 && wave == (int)((Kw / WaveKCfg::KC) % waves);
    int64_t k0 = (int64_t)wave * WaveKCfg::KC;
    if (tail) {
        opa.load_tail(r.a, Kw, left, lane);
        opb.load_tail(r.b, Kw, left, lane);
        k0 -= step;   // counts as the chunk before the first
    } else if (k0 < Kw) {
        load(k0);
    }
    // Staged, its registers refilled, multiplied: the next chunk's loads are in flight under this one's MFMAs and
    // the other waves'.  (Two register sets, two chunks ahead, were 5-12 % slower on every product tried and did
    // not fit the 4 x 4 tile of two K-contiguous operands.)
    for (; k0 < Kw; k0 += step) {
        stage();
        if (k0 + step < Kw) load(k0 + step);
        multiply_half(0);
        if (k0 >= 0 || left > 32) multiply_half(1);   // the second half of a tail of up to 32 k is zeros
        wave_order();
    }

    // this lane's four outputs of block (i, j): C[m][n .. n + 3]
    auto store = [&](int i, int j, const f32x4& v) __attribute__((always_inline)) {
        const int64_t m = m0 + 16 * i + (lane & 15), n = n0 + 16 * j + 4 * (lane >> 4);
        if (m >= M || n >= N) return;
        uint16_t* pc = C + m * ldc + n;
        const u32x2 w{pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
        if (n + 4 <= N) {
            *reinterpret_cast<u32x2_any*>(pc) = w;
        } else {
            pc[0] = (uint16_t)(w[0] & 0xFFFFu);
            if (n + 1 < N) pc[1] = (uint16_t)(w[0] >> 16);
            if (n + 2 < N) pc[2] = (uint16_t)(w[1] & 0xFFFFu);
        }
    };
    if (waves == 1) {
        // the only wave of the tile: through its LDS region, a block row at a time, to 16-byte stores of whole rows
        if (NI >= 2 && m0 + TM <= M && n0 + TN <= N) {
            constexpr int CPR = TN / 8;   // 16-byte pieces per row
#pragma unroll
            for (int i = 0; i < MI; ++i) {
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    *reinterpret_cast<u32x2*>(smem + (lane & 15) * (2 * TN + 16) + 32 * j + 8 * (lane >> 4)) =
                        u32x2{pack2_bf16(acc[i][j][0], acc[i][j][1]), pack2_bf16(acc[i][j][2], acc[i][j][3])};
                wave_order();
#pragma unroll
                for (int it = 0; it < 16 * CPR / 64; ++it) {
                    const int q = it * 64 + lane, r = q / CPR, ch = q % CPR;
                    const u32x4 v = *reinterpret_cast<const u32x4*>(smem + r * (2 * TN + 16) + 16 * ch);
                    *reinterpret_cast<u32x4_any*>(C + (m0 + 16 * i + r) * ldc + n0 + 8 * ch) = v;
                }
                wave_order();
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) store(i, j, acc[i][j]);
        return;
    }
    // partial tiles to LDS, 1 KB per (wave, block); then wave w adds up the blocks w, w + waves, ... over the
    // waves in their order
    __syncthreads();   // the staging regions are free
    f32x4* const part = reinterpret_cast<f32x4*>(smem);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) part[((wave * MI + i) * NI + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    for (int b = wave; b < MI * NI; b += waves) {
        f32x4 v = part[b * 64 + lane];
        for (int w = 1; w < waves; ++w) v += part[(w * (MI * NI) + b) * 64 + lane];
        store(b / NI, b % NI, v);
    }
}

// The weight gradient of a few tokens: two MN-contiguous operands over K <= 32 H (H = 1, 2), M >= 64, N >= 64.  All of K is one
// chunk, so what counts is the output, written once, and how many waves are there to write it.  A workgroup of
// four waves takes 64 rows and, SPAN times, 4 x 64 columns (a wave whose columns would all be another's has no work); a wave's region of LDS holds 32 H k-rows (wave-K kernel: 64 of
// both operands), the fragments of the rows stay in registers, the next columns' loads are in flight while 16 rows at a time
// are multiplied, rounded and stored as whole lines.  Products and sums are the wave-K kernel's, to the bit.
// What bounds it is the output's way to memory.  On the wave-K kernel eight waves fit a compute unit's LDS (18 KB each) and
// each lived for one tile: load, multiply, store.  us, before / here: 2048 x 8192 x 24 11.8 / 8.9 (clearing the output: 7.6), x 64
// 11.5 / 9.9, 4096 x 16384 x 48 from HBM 53 / 31, 1024 x 4096 x 24 6.2 / 4.7, 2001 x 8191 x 31 12.5 / 10.1.
struct ShortKCfg {
    static constexpr int ROWB = 32 * 4 + WaveKCfg::PAD;            // bytes per k-row, or output row, in LDS
    static constexpr int COLS = 4 * 64;                             // per workgroup and step
    static constexpr int wave_bytes(int H) { return 32 * H * ROWB + 16 * ROWB; }
};
template <int H, bool CHUNKS>
__global__ __launch_bounds__(256, (H == 1 ? 4 : 3)) void gemm_shortk_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, uint16_t* __restrict__ C,
                                                          int64_t M, int64_t N, int K, int64_t lda, int64_t ldb, int64_t ldc, int tiles_n, int span) {
    constexpr int ROWB = ShortKCfg::ROWB, NL = 4 * H;
    __shared__ __attribute__((aligned(16))) uint8_t smem[4 * ShortKCfg::wave_bytes(H)];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* const region = smem + wave * ShortKCfg::wave_bytes(H);
    uint8_t* const rows16 = region + 32 * H * ROWB;
    const int spans = (tiles_n + span - 1) / span;   // tiles_n: steps of COLS columns
    int id = blockIdx.x;
    if constexpr (CHUNKS) {   // XCD x runs the workgroups x, x + 8, ...: a contiguous chunk of the sequence
        const uint32_t x = blockIdx.x & 7, rem = gridDim.x & 7;
        id = (int)(x * (gridDim.x >> 3) + min(x, rem) + (blockIdx.x >> 3));
    }
    const int tile_m = id / spans, first = (id - tile_m * spans) * span, last = min(first + span, tiles_n);
    const int64_t m0 = min((int64_t)tile_m * 64, M - 64);
    // columns from N on are another wave's; there is no barrier in this kernel
    const int mine = (int)min((int64_t)last, (N - 64 * wave + ShortKCfg::COLS - 1) / ShortKCfg::COLS);
    if (first >= mine) return;

    // a load is 8 k-rows x 128 bytes; k-rows behind K: the last one again, dropped
    const int kr = lane >> 3, ch = lane & 7;
    const auto load = [&](u32x4 (&x)[NL], const uint16_t* P, int64_t ld) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NL; ++j)
            if (8 * j < K) x[j] = *reinterpret_cast<const u32x4_any*>(P + min(8 * j + kr, K - 1) * ld + 8 * ch);
    };
    const auto stage = [&](const u32x4 (&x)[NL]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NL; ++j)
            *reinterpret_cast<u32x4*>(region + (8 * j + kr) * ROWB + 16 * ch) = 8 * j + kr < K ? x[j] : u32x4{0u, 0u, 0u, 0u};
        wave_order();
    };
    const auto fragments = [&](bf16x8 (&f)[4][H]) __attribute__((always_inline)) {
        typedef short i16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
        const int s = lane & 15, g = lane >> 4;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const uint8_t* const p = region + (32 * h + 8 * g + (s >> 2)) * ROWB + 8 * (s & 3) + 32 * b;
                const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p));
                const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + 4 * ROWB));
                f[b][h] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        wave_order();
    };
    const auto column = [&](int tile) __attribute__((always_inline)) { return min((int64_t)tile * ShortKCfg::COLS + 64 * wave, N - 64); };

    u32x4 xa[NL] = {}, xb[NL] = {};
    bf16x8 fa[4][H], fb[4][H];
    load(xa, A + m0, lda);
    load(xb, B + column(first), ldb);
    stage(xa);
    fragments(fa);
    for (int tile = first; tile < mine; ++tile) {
        const int64_t n0 = column(tile);
        stage(xb);
        if (tile + 1 < mine) load(xb, B + column(tile + 1), ldb);
        fragments(fb);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int h = 0; h < H; ++h) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][h], fa[i][h], acc, 0, 0, 0);
                *reinterpret_cast<u32x2*>(rows16 + (lane & 15) * ROWB + 32 * j + 8 * (lane >> 4)) = u32x2{pack2_bf16(acc[0], acc[1]), pack2_bf16(acc[2], acc[3])};
            }
            wave_order();
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(rows16 + (8 * it + kr) * ROWB + 16 * ch);
                *reinterpret_cast<u32x4_any*>(C + (m0 + 16 * i + 8 * it + kr) * ldc + n0 + 8 * ch) = v;
            }
            wave_order();
        }
    }
}

}  // namespace axonn
