// Translation unit of the smaller tiles on the 32-k LDS ring (see kernels.hpp).
#include "kernels.hpp"
#include "gemm_mfma16.hpp"

namespace axonn {

#define AXONN_RING3(BM, BN, ...)                                                        \
    {gemm_tile_kernel16<BM, BN, 2, 2, true, false, __VA_ARGS__>, gemm_tile_kernel16<BM, BN, 2, 2, true, true, __VA_ARGS__>, \
     gemm_tile_kernel16<BM, BN, 2, 2, false, false, __VA_ARGS__>}

#define AXONN_RING2(BM, BN, ...)                                                        \
    {gemm_tile_kernel16<BM, BN, 2, 2, true, false, __VA_ARGS__>, nullptr, gemm_tile_kernel16<BM, BN, 2, 2, false, false, __VA_ARGS__>}

// Without split-K the eight-wave kernel is ahead on all these tiles (gemm_mfma16_k64g.hpp); one form is left, under the name
// of the variant that plans of 128 large tiles carry.
tile_kernel_t ring_kernel_small(int bm, int bn, bool split, int layout) {
    static const tile_kernel_t k128x256[3] = AXONN_RING3(128, 256, false);
    static const tile_kernel_t k256x128_sk[3] = AXONN_RING3(256, 128, true);
    static const tile_kernel_t k128x256_sk[3] = AXONN_RING3(128, 256, true);
    // two K-contiguous operands (NT): the 64-k kernel has that tile (k64_kernel_half)
    static const tile_kernel_t k128x128_sk[3] = AXONN_RING2(128, 128, true);
    if (layout < 0 || layout > 2) return nullptr;
    if (bm == 128 && bn == 256) return (split ? k128x256_sk : k128x256)[layout];
    if (bm == 256 && bn == 128 && split) return k256x128_sk[layout];
    if (bm == 128 && bn == 128 && split) return k128x128_sk[layout];
    return nullptr;
}

}  // namespace axonn
