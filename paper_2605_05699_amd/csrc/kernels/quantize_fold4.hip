// Write path at d = 256, folded twice (a quarter of the dense matrix work): 4- and 8-bit codes, g = 16, 32 and 256, and the
// abs-max statistic.
#include "../quantize_fold4_tiles.h"

namespace {
template <int BITS>
quantize_kernel_t pick(int gm) {
    return gm == kGroup16 ? srft_quantize_fold4_kernel<BITS, kGroup16>
         : gm == kGroupWide ? srft_quantize_fold4_kernel<BITS, kGroupWide> : srft_quantize_fold4_kernel<BITS, kGroup32>;
}
template <int BITS>
batched_kernels_t pick_batched(int gm) {
    return gm == kGroup16 ? SRFT_BATCHED(srft_quantize_fold4_batched_kernel, BITS, kGroup16)
         : gm == kGroupWide ? SRFT_BATCHED(srft_quantize_fold4_batched_kernel, BITS, kGroupWide)
                            : SRFT_BATCHED(srft_quantize_fold4_batched_kernel, BITS, kGroup32);
}
}  // namespace

quantize_kernel_t srft_pick_quantize_fold4(int bits, int gm) { return bits == 8 ? pick<8>(gm) : pick<4>(gm); }
quantize_kernel_t srft_pick_quantize_fold4_amax(int teams) {
    return teams == 1 ? srft_quantize_fold4_amax_kernel<1> : teams == 2 ? srft_quantize_fold4_amax_kernel<2> : nullptr;
}
batched_kernels_t srft_pick_quantize_fold4_batched(int bits, int gm) { return bits == 8 ? pick_batched<8>(gm) : pick_batched<4>(gm); }
int srft_fold4_table_units(void) { return kFold4Units; }
