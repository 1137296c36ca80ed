// Read path, twice-folded form (d = 128 and 256 at g >= 32, d = 256 at g = 16), 4- and 8-bit codes.
#include "../dequantize_fold4_tiles.h"

dequantize_kernel_t srft_pick_dequantize_fold4(int d, int bits, bool fine) {
    if (fine) return d != 256 ? nullptr : bits == 8 ? srft_dequantize_fold4_kernel<256, 8, true> : srft_dequantize_fold4_kernel<256, 4, true>;
    if (d == 128) return bits == 8 ? srft_dequantize_fold4_kernel<128, 8, false> : srft_dequantize_fold4_kernel<128, 4, false>;
    if (d == 256) return bits == 8 ? srft_dequantize_fold4_kernel<256, 8, false> : srft_dequantize_fold4_kernel<256, 4, false>;
    return nullptr;
}
batched_kernels_t srft_pick_dequantize_fold4_batched(int d, int bits, bool fine) {
    if (fine && d != 256) return nullptr;
    if (fine) return bits == 8 ? SRFT_BATCHED(srft_dequantize_fold4_batched_kernel, 256, 8, true) : SRFT_BATCHED(srft_dequantize_fold4_batched_kernel, 256, 4, true);
    if (d == 128) return bits == 8 ? SRFT_BATCHED(srft_dequantize_fold4_batched_kernel, 128, 8, false) : SRFT_BATCHED(srft_dequantize_fold4_batched_kernel, 128, 4, false);
    if (d == 256) return bits == 8 ? SRFT_BATCHED(srft_dequantize_fold4_batched_kernel, 256, 8, false) : SRFT_BATCHED(srft_dequantize_fold4_batched_kernel, 256, 4, false);
    return nullptr;
}
int srft_rfold4_table_units(int d) { return srft_rfold4_units(d); }
