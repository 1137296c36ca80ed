// Write path, plain form, 8-bit codes: every (d, group mode, way of the record) instance.
#include "../quantize_tiles.h"

namespace {
template <int D, int S, bool STAGED>
quantize_kernel_t by_group_mode(int gm) {
    switch (gm) {
        case kGroup16: return srft_quantize_kernel<D, S, kOutCodes, kGroup16, 8, STAGED>;
        case kGroupWide: return srft_quantize_kernel<D, S, kOutCodes, kGroupWide, 8, STAGED>;
        default: return srft_quantize_kernel<D, S, kOutCodes, kGroup32, 8, STAGED>;
    }
}
template <int D>
quantize_kernel_t pick(int gm, bool staged) {
    constexpr int S = D == 64 ? 2 : 1;
    return staged ? by_group_mode<D, S, D != 32>(gm) : by_group_mode<D, S, false>(gm);      // (d = 32: srft_write_staged)
}
template <int D, int S, bool STAGED>
batched_kernels_t batched_by_group_mode(int gm) {
    return gm == kGroup16 ? SRFT_BATCHED(srft_quantize_batched_kernel, D, S, kGroup16, 8, STAGED)
         : gm == kGroupWide ? SRFT_BATCHED(srft_quantize_batched_kernel, D, S, kGroupWide, 8, STAGED)
                            : SRFT_BATCHED(srft_quantize_batched_kernel, D, S, kGroup32, 8, STAGED);
}
template <int D>
batched_kernels_t pick_batched(int gm, bool staged) {
    constexpr int S = D == 64 ? 2 : 1;
    return staged ? batched_by_group_mode<D, S, D != 32>(gm) : batched_by_group_mode<D, S, false>(gm);      // (d = 32: srft_write_staged)
}
}  // namespace

quantize_kernel_t srft_pick_quantize_plain_b8(int d, int gm, bool staged) { SRFT_DISPATCH_D(d, pick, gm, staged) }
batched_kernels_t srft_pick_quantize_plain_batched_b8(int d, int gm, bool staged) {
    SRFT_DISPATCH_D(d, pick_batched, gm, staged)
}
