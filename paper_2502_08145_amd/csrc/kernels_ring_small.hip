// Translation unit of the smaller tiles on the 32-k LDS ring (see kernels.hpp).
#include "kernels.hpp"
#include "gemm_mfma16.hpp"

namespace axonn {

#define AXONN_RING3(BM, BN, WN, ...)                                                        \
    {gemm_tile_kernel16<BM, BN, 2, WN, true, false, __VA_ARGS__>, gemm_tile_kernel16<BM, BN, 2, WN, true, true, __VA_ARGS__>, \
     gemm_tile_kernel16<BM, BN, 2, WN, false, false, __VA_ARGS__>}

#define AXONN_RING2(BM, BN, WN, ...)                                                        \
    {gemm_tile_kernel16<BM, BN, 2, WN, true, false, __VA_ARGS__>, nullptr, gemm_tile_kernel16<BM, BN, 2, WN, false, false, __VA_ARGS__>}

tile_kernel_t ring_kernel_small(int bm, int bn, int wn, bool split, int layout, bool k_tail) {
    static const tile_kernel_t k256x128[3] = AXONN_RING3(256, 128, 2, false);
    static const tile_kernel_t k128x256[3] = AXONN_RING3(128, 256, 2, false);
    static const tile_kernel_t k128x256_w8[3] = AXONN_RING3(128, 256, 4, false);
    static const tile_kernel_t k256x128_sk[3] = AXONN_RING3(256, 128, 2, true);
    static const tile_kernel_t k128x256_sk[3] = AXONN_RING3(128, 256, 2, true);
    // two K-contiguous operands (NT): the 64-k kernel has that tile (k64_kernel_half)
    static const tile_kernel_t k128x128[3] = AXONN_RING2(128, 128, 2, false);
    static const tile_kernel_t k128x128_sk[3] = AXONN_RING2(128, 128, 2, true);
    // ... and is ahead on the half tiles, so no plan of a ragged K leaves NT here
    static const tile_kernel_t k256x128_tail[3] = AXONN_RING2(256, 128, 2, false, true);
    static const tile_kernel_t k128x256_w8_tail[3] = AXONN_RING2(128, 256, 4, false, true);
    static const tile_kernel_t k128x128_tail[3] = AXONN_RING2(128, 128, 2, false, true);
    if (layout < 0 || layout > 2) return nullptr;
    if (k_tail) {
        if (split) return nullptr;
        if (bm == 256 && bn == 128 && wn == 2) return k256x128_tail[layout];
        if (bm == 128 && bn == 256 && wn == 4) return k128x256_w8_tail[layout];
        if (bm == 128 && bn == 128 && wn == 2) return k128x128_tail[layout];
        return nullptr;
    }
    if (bm == 256 && bn == 128 && wn == 2) return (split ? k256x128_sk : k256x128)[layout];
    if (bm == 128 && bn == 256 && wn == 2) return (split ? k128x256_sk : k128x256)[layout];
    if (bm == 128 && bn == 256 && wn == 4 && !split) return k128x256_w8[layout];
    if (bm == 128 && bn == 128 && wn == 2) return (split ? k128x128_sk : k128x128)[layout];
    return nullptr;
}

}  // namespace axonn
