// Read path, 8-bit codes: every (d, slabs per wavefront, group mode) instance; d = 192 folded, the others plain (d = 128 and 256 run
// the twice-folded kernel, except with Hadamard and at d = 128, g = 16).  Each with the rows written through or left to the L2.
#include "../dequantize_tiles.h"

namespace {
template <int D, bool THROUGH>
dequantize_kernel_t pick_way(int slabs, int gm) {
    if constexpr (D == 192) {
        return gm == kGroup16 ? srft_dequantize_kernel<D, 2, 2, true, 8, THROUGH> : srft_dequantize_kernel<D, 2, 1, true, 8, THROUGH>;
    } else {
        if constexpr (D == 64)
            if (slabs == 2) return gm == kGroup16 ? srft_dequantize_kernel<D, 2, 1, false, 8, THROUGH> : srft_dequantize_kernel<D, 2, 2, false, 8, THROUGH>;
        return gm == kGroup16 ? srft_dequantize_kernel<D, 1, 1, false, 8, THROUGH> : srft_dequantize_kernel<D, 1, 2, false, 8, THROUGH>;
    }
}
template <int D, bool THROUGH>
batched_kernels_t pick_batched_way(int slabs, int gm) {
    if constexpr (D == 192) {
        return gm == kGroup16 ? SRFT_BATCHED(srft_dequantize_batched_kernel, D, 2, 2, true, 8, THROUGH) : SRFT_BATCHED(srft_dequantize_batched_kernel, D, 2, 1, true, 8, THROUGH);
    } else {
        if constexpr (D == 64)
            if (slabs == 2) return gm == kGroup16 ? SRFT_BATCHED(srft_dequantize_batched_kernel, D, 2, 1, false, 8, THROUGH) : SRFT_BATCHED(srft_dequantize_batched_kernel, D, 2, 2, false, 8, THROUGH);
        return gm == kGroup16 ? SRFT_BATCHED(srft_dequantize_batched_kernel, D, 1, 1, false, 8, THROUGH) : SRFT_BATCHED(srft_dequantize_batched_kernel, D, 1, 2, false, 8, THROUGH);
    }
}
template <int D>
dequantize_kernel_t pick(int slabs, int gm, bool through) {
    return through ? pick_way<D, true>(slabs, gm) : pick_way<D, false>(slabs, gm);
}
template <int D>
batched_kernels_t pick_batched(int slabs, int gm, bool through) {
    return through ? pick_batched_way<D, true>(slabs, gm) : pick_batched_way<D, false>(slabs, gm);
}
}  // namespace

dequantize_kernel_t srft_pick_dequantize_b8(int d, int slabs, int gm, bool through) {
    SRFT_DISPATCH_D(d, pick, slabs, gm, through)
}
batched_kernels_t srft_pick_dequantize_batched_b8(int d, int slabs, int gm, bool through) {
    SRFT_DISPATCH_D(d, pick_batched, slabs, gm, through)
}
