// Translation unit of the smaller tiles on the 32-k LDS ring (see kernels.hpp).
#include "kernels.hpp"
#include "gemm_mfma16.hpp"

namespace axonn {

#define AXONN_RING(BM, BN, A_KC, B_KC) gemm_tile_kernel16<BM, BN, 2, 2, A_KC, B_KC, true>
#define AXONN_RING3(BM, BN) {AXONN_RING(BM, BN, true, false), AXONN_RING(BM, BN, true, true), AXONN_RING(BM, BN, false, false)}

// With split-K only: without it the eight-wave kernel is ahead on all these tiles (gemm_mfma16_k64g.hpp).
tile_kernel_t ring_kernel_small(int bm, int bn, int layout) {
    static const tile_kernel_t k256x128[3] = AXONN_RING3(256, 128);
    static const tile_kernel_t k128x256[3] = AXONN_RING3(128, 256);
    // two K-contiguous operands (NT): the 64-k kernel has that tile (k64_kernel_half)
    static const tile_kernel_t k128x128[3] = {AXONN_RING(128, 128, true, false), nullptr, AXONN_RING(128, 128, false, false)};
    if (layout < 0 || layout > 2) return nullptr;
    if (bm == 256 && bn == 128) return k256x128[layout];
    if (bm == 128 && bn == 256) return k128x256[layout];
    if (bm == 128 && bn == 128) return k128x128[layout];
    return nullptr;
}

}  // namespace axonn
