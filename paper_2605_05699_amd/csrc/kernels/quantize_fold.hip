// Write path, folded form: d = 128, 4- and 8-bit codes, g = 32 or wider groups; d = 256, g = 64 and 128.  Each with the record written
// through or left to the L2.
#include "../quantize_fold_tiles.h"

namespace {
template <int D, bool THROUGH>
quantize_kernel_t pick(int bits, bool wide) {
    if constexpr (D != 256) {
        if (!wide) return bits == 8 ? srft_quantize_fold_kernel<D, 8, false, THROUGH> : srft_quantize_fold_kernel<D, 4, false, THROUGH>;
    }
    return bits == 8 ? srft_quantize_fold_kernel<D, 8, true, THROUGH> : srft_quantize_fold_kernel<D, 4, true, THROUGH>;
}
template <int D, bool THROUGH>
batched_kernels_t pick_batched(int bits, bool wide) {
    if constexpr (D != 256) {
        if (!wide)
            return bits == 8 ? SRFT_BATCHED(srft_quantize_fold_batched_kernel, D, 8, false, THROUGH)
                             : SRFT_BATCHED(srft_quantize_fold_batched_kernel, D, 4, false, THROUGH);
    }
    return bits == 8 ? SRFT_BATCHED(srft_quantize_fold_batched_kernel, D, 8, true, THROUGH)
                     : SRFT_BATCHED(srft_quantize_fold_batched_kernel, D, 4, true, THROUGH);
}
}  // namespace

quantize_kernel_t srft_pick_quantize_fold(int d, int bits, bool wide, bool through) {
    return d == 128 ? (through ? pick<128, true>(bits, wide) : pick<128, false>(bits, wide))
           : d == 256 ? (through ? pick<256, true>(bits, wide) : pick<256, false>(bits, wide))
                      : nullptr;
}
quantize_kernel_t srft_pick_quantize_fold_amax(int teams) {
    return teams == 1   ? srft_quantize_fold_amax_kernel<128, 1>
           : teams == 2 ? srft_quantize_fold_amax_kernel<128, 2>
           : teams == 4 ? srft_quantize_fold_amax_kernel<128, 4>
                        : nullptr;
}
batched_kernels_t srft_pick_quantize_fold_batched(int d, int bits, bool wide, bool through) {
    return d == 128 ? (through ? pick_batched<128, true>(bits, wide) : pick_batched<128, false>(bits, wide))
           : d == 256 ? (through ? pick_batched<256, true>(bits, wide) : pick_batched<256, false>(bits, wide))
                      : nullptr;
}
