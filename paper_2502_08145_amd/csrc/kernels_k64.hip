// Translation unit of the 256 x 256 tile kernels with 64-k LDS stages (see kernels.hpp).
#include "kernels.hpp"
#include "gemm_mfma16_k64.hpp"
#include "gemm_mfma16_k64p.hpp"

namespace axonn {

// Load schedule per mode (see gemm_tile_kernel_k64): with two K-contiguous operands (NT) the A panel is
// triple-buffered and fetched in sub-step 0, measured 3-5 % faster at K of 4096 and more (2048 x 16384 x 4096:
// 1320 -> 1390 TFLOP/s, 8192^3: 1465 -> 1512) and no slower elsewhere; with an MN-contiguous operand it
// makes no difference (NN) or costs 2-5 % (TN, either operand triple-buffered), so those keep two buffers each.
constexpr int kSchedNN = 0, kSchedNT = 1, kSchedTN = 0;

tile_kernel_t k64_kernel(bool split, int layout, bool k_tail) {
    if (k_tail) {
        static const tile_kernel_t tail[3] = {gemm_tile_kernel_k64<256, 256, 4, true, false, false, kSchedNN, true>,
                                              gemm_tile_kernel_k64<256, 256, 4, true, true, false, kSchedNT, true>,
                                              gemm_tile_kernel_k64<256, 256, 4, false, false, false, kSchedTN, true>};
        return (!split && layout >= 0 && layout < 3) ? tail[layout] : nullptr;
    }
    static const tile_kernel_t fn[2][3] = {
        {gemm_tile_kernel_k64<256, 256, 4, true, false, false, kSchedNN>, gemm_tile_kernel_k64<256, 256, 4, true, true, false, kSchedNT>,
         gemm_tile_kernel_k64<256, 256, 4, false, false, false, kSchedTN>},
        {gemm_tile_kernel_k64<256, 256, 4, true, false, true, kSchedNN>, gemm_tile_kernel_k64<256, 256, 4, true, true, true, kSchedNT>,
         gemm_tile_kernel_k64<256, 256, 4, false, false, true, kSchedTN>},
    };
    return (layout >= 0 && layout < 3) ? fn[split ? 1 : 0][layout] : nullptr;
}

// The 64-k kernel on the half tiles: four waves (2 x 2), three buffers per operand (144 KB), half of an
// iteration's loads in either sub-step.  NT only: there it measures 28 % over the 32-k ring on the same
// tiles (2048 x 4096 x 4096: 1018 against 794 TFLOP/s; 4096^3: 1141 against 949); with an MN-contiguous
// operand it is 15-30 % BEHIND the ring (NN 743 against 990, TN 704 against 904), like every schedule
// tried that issues such an operand's loads anywhere but straight after the barrier.  128 x 128 tiles (96 KB, four
// waves) gain less, but gain at every size: alternating runs against the ring, one product of 2048 x 2048 x 8192
// 73.0 -> 65.8 us (operands from HBM 87 -> 81), 1024 x 3072 x 3072 29.6 -> 27.1 (39.2 -> 37.4), 2048 x 640 x 640 from HBM 9.0 ->
// 8.0: every load is a whole line and there is one barrier per 64 k; their bytes in flight do not matter (the
// ring with eight stages instead of six: no change).
tile_kernel_t k64_kernel_half(int bm, int bn, bool split, int layout, bool k_tail) {
    if (layout != 1 || (split && k_tail)) return nullptr;
    if (bm == 128 && bn == 128)
        return split    ? gemm_tile_kernel_k64<128, 128, 2, true, true, true, 3>
               : k_tail ? gemm_tile_kernel_k64<128, 128, 2, true, true, false, 3, true>
                        : gemm_tile_kernel_k64<128, 128, 2, true, true, false, 3>;
    if (k_tail && bm == 256 && bn == 128) return gemm_tile_kernel_k64<256, 128, 2, true, true, false, 3, true>;
    if (k_tail && bm == 128 && bn == 256) return gemm_tile_kernel_k64<128, 256, 2, true, true, false, 3, true>;
    if (bm == 256 && bn == 128)
        return split ? gemm_tile_kernel_k64<256, 128, 2, true, true, true, 3> : gemm_tile_kernel_k64<256, 128, 2, true, true, false, 3>;
    if (bm == 128 && bn == 256)
        return split ? gemm_tile_kernel_k64<128, 256, 2, true, true, true, 3> : gemm_tile_kernel_k64<128, 256, 2, true, true, false, 3>;
    return nullptr;
}

tile_kernel_t k64p_kernel(int layout) {
    static const tile_kernel_t fn[3] = {gemm_tile_kernel_k64p<true, false>, gemm_tile_kernel_k64p<true, true>,
                                        gemm_tile_kernel_k64p<false, false>};
    return (layout >= 0 && layout < 3) ? fn[layout] : nullptr;
}

}  // namespace axonn
