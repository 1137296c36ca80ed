// A cache's flush: the folded forms of the write path (d = 128 and 256), alone and with the twice-folded read path behind them.
#include "../cache_flush.h"

namespace {
template <int D, int BITS, class WRITE, bool FINE = false>
flush_kernels_t kernels() {
    return {srft_cache_flush_kernel<D, D, WRITE, srft_flush_read_later>, srft_cache_flush_kernel<D, D, WRITE, srft_flush_read_fold4<D, BITS, FINE>>};
}
template <int BITS>
flush_kernels_t pick(int d, int gm, bool fold4_q) {
    if (d == 128)
        return gm == kGroupWide ? kernels<128, BITS, srft_flush_write_fold<128, BITS, true>>() : kernels<128, BITS, srft_flush_write_fold<128, BITS, false>>();
    if (d != 256) return nullptr;
    if (!fold4_q) return kernels<256, BITS, srft_flush_write_fold<256, BITS, true>>();
    if (gm == kGroup16) return kernels<256, BITS, srft_flush_write_fold4<BITS, kGroup16>, true>();
    return gm == kGroupWide ? kernels<256, BITS, srft_flush_write_fold4<BITS, kGroupWide>>() : kernels<256, BITS, srft_flush_write_fold4<BITS, kGroup32>>();
}
}  // namespace

flush_kernels_t srft_pick_cache_flush_fold(int d, int bits, int gm, bool fold4_q) {
    return bits == 8 ? pick<8>(d, gm, fold4_q) : pick<4>(d, gm, fold4_q);
}
