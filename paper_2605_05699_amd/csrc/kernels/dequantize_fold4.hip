// Read path, twice-folded form (d = 128 and 256 at g >= 32, d = 256 at g = 16), 4- and 8-bit codes.  Each with the rows written through
// or left to the L2.
#include "../dequantize_fold4_tiles.h"

namespace {
template <bool THROUGH>
dequantize_kernel_t pick(int d, int bits, bool fine) {
    if (fine) return d != 256 ? nullptr : bits == 8 ? srft_dequantize_fold4_kernel<256, 8, true, THROUGH> : srft_dequantize_fold4_kernel<256, 4, true, THROUGH>;
    if (d == 128) return bits == 8 ? srft_dequantize_fold4_kernel<128, 8, false, THROUGH> : srft_dequantize_fold4_kernel<128, 4, false, THROUGH>;
    if (d == 256) return bits == 8 ? srft_dequantize_fold4_kernel<256, 8, false, THROUGH> : srft_dequantize_fold4_kernel<256, 4, false, THROUGH>;
    return nullptr;
}
template <int D, bool FINE, bool THROUGH>
batched_kernels_t batched(int bits) {
    return bits == 8 ? SRFT_BATCHED(srft_dequantize_fold4_batched_kernel, D, 8, FINE, THROUGH)
                     : SRFT_BATCHED(srft_dequantize_fold4_batched_kernel, D, 4, FINE, THROUGH);
}
template <bool THROUGH>
batched_kernels_t pick_batched(int d, int bits, bool fine) {
    if (fine) return d == 256 ? batched<256, true, THROUGH>(bits) : nullptr;
    return d == 128 ? batched<128, false, THROUGH>(bits) : d == 256 ? batched<256, false, THROUGH>(bits) : nullptr;
}
}  // namespace

dequantize_kernel_t srft_pick_dequantize_fold4(int d, int bits, bool fine, bool through) {
    return through ? pick<true>(d, bits, fine) : pick<false>(d, bits, fine);
}
batched_kernels_t srft_pick_dequantize_fold4_batched(int d, int bits, bool fine, bool through) {
    return through ? pick_batched<true>(d, bits, fine) : pick_batched<false>(d, bits, fine);
}
int srft_rfold4_table_units(int d) { return srft_rfold4_units(d); }
