// Read path, 8-bit codes: every (d, slabs per wavefront, group mode) instance; d = 192 folded, the others plain (d = 128 and 256 run
// the twice-folded kernel, except with Hadamard and at d = 128, g = 16).
#include "../dequantize_tiles.h"

namespace {
template <int D>
dequantize_kernel_t pick(int slabs, int gm) {
    if constexpr (D == 192) {
        return gm == kGroup16 ? srft_dequantize_kernel<D, 2, 2, true, 8> : srft_dequantize_kernel<D, 2, 1, true, 8>;
    } else {
        if constexpr (D == 64)
            if (slabs == 2) return gm == kGroup16 ? srft_dequantize_kernel<D, 2, 1, false, 8> : srft_dequantize_kernel<D, 2, 2, false, 8>;
        return gm == kGroup16 ? srft_dequantize_kernel<D, 1, 1, false, 8> : srft_dequantize_kernel<D, 1, 2, false, 8>;
    }
}
template <int D>
batched_kernels_t pick_batched(int slabs, int gm) {
    if constexpr (D == 192) {
        return gm == kGroup16 ? SRFT_BATCHED(srft_dequantize_batched_kernel, D, 2, 2, true, 8) : SRFT_BATCHED(srft_dequantize_batched_kernel, D, 2, 1, true, 8);
    } else {
        if constexpr (D == 64)
            if (slabs == 2) return gm == kGroup16 ? SRFT_BATCHED(srft_dequantize_batched_kernel, D, 2, 1, false, 8) : SRFT_BATCHED(srft_dequantize_batched_kernel, D, 2, 2, false, 8);
        return gm == kGroup16 ? SRFT_BATCHED(srft_dequantize_batched_kernel, D, 1, 1, false, 8) : SRFT_BATCHED(srft_dequantize_batched_kernel, D, 1, 2, false, 8);
    }
}
}  // namespace

dequantize_kernel_t srft_pick_dequantize_b8(int d, int slabs, int gm) {
    SRFT_DISPATCH_D(d, pick, slabs, gm)
}
batched_kernels_t srft_pick_dequantize_batched_b8(int d, int slabs, int gm) {
    SRFT_DISPATCH_D(d, pick_batched, slabs, gm)
}
