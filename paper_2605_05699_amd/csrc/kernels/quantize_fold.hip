// Write path, folded form: d = 128, 4- and 8-bit codes, g = 32 or wider groups; d = 256, g = 64 and 128.
#include "../quantize_fold_tiles.h"

namespace {
template <int D>
quantize_kernel_t pick(int bits, bool wide) {
    if constexpr (D != 256) {
        if (!wide) return bits == 8 ? srft_quantize_fold_kernel<D, 8, false> : srft_quantize_fold_kernel<D, 4, false>;
    }
    return bits == 8 ? srft_quantize_fold_kernel<D, 8, true> : srft_quantize_fold_kernel<D, 4, true>;
}
template <int D>
batched_kernels_t pick_batched(int bits, bool wide) {
    if constexpr (D != 256) {
        if (!wide)
            return bits == 8 ? SRFT_BATCHED(srft_quantize_fold_batched_kernel, D, 8, false) : SRFT_BATCHED(srft_quantize_fold_batched_kernel, D, 4, false);
    }
    return bits == 8 ? SRFT_BATCHED(srft_quantize_fold_batched_kernel, D, 8, true) : SRFT_BATCHED(srft_quantize_fold_batched_kernel, D, 4, true);
}
}  // namespace

quantize_kernel_t srft_pick_quantize_fold(int d, int bits, bool wide) {
    return d == 128 ? pick<128>(bits, wide) : d == 256 ? pick<256>(bits, wide) : nullptr;
}
quantize_kernel_t srft_pick_quantize_fold_amax(int teams) {
    return teams == 1   ? srft_quantize_fold_amax_kernel<128, 1>
           : teams == 2 ? srft_quantize_fold_amax_kernel<128, 2>
           : teams == 4 ? srft_quantize_fold_amax_kernel<128, 4>
                        : nullptr;
}
batched_kernels_t srft_pick_quantize_fold_batched(int d, int bits, bool wide) {
    return d == 128 ? pick_batched<128>(bits, wide) : d == 256 ? pick_batched<256>(bits, wide) : nullptr;
}
