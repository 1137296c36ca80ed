// A cache's flush: the plain form of the write path, alone and with the plain form of the read path behind it.
#include "../cache_flush.h"

namespace {
template <int D, int S, int GM, int BITS>
flush_kernels_t kernels() {
    constexpr int NT = 2 * D / S, KS = GM == kGroup16 ? 1 : 2;
    const auto alone = srft_cache_flush_kernel<D, NT, srft_flush_write_plain<D, S, GM, BITS, D != 32>, srft_flush_read_later>;
    if constexpr (D <= 128)
        return {alone, srft_cache_flush_kernel<D, NT, srft_flush_write_plain<D, S, GM, BITS, false>, srft_flush_read_plain<D, S, KS, BITS>>};
    else
        return {alone, nullptr};
}
template <int D>
flush_kernels_t pick(int bits, int gm) {
    constexpr int S = D == 64 ? 2 : 1;
    if (bits == 8)
        return gm == kGroup16 ? kernels<D, S, kGroup16, 8>() : gm == kGroupWide ? kernels<D, S, kGroupWide, 8>() : kernels<D, S, kGroup32, 8>();
    return gm == kGroup16 ? kernels<D, S, kGroup16, 4>() : gm == kGroupWide ? kernels<D, S, kGroupWide, 4>() : kernels<D, S, kGroup32, 4>();
}
flush_kernels_t dispatch(int d, int bits, int gm) {
    SRFT_DISPATCH_D(d, pick, bits, gm)
}
}  // namespace

flush_kernels_t srft_pick_cache_flush_plain(int d, int bits, int gm) { return dispatch(d, bits, gm); }
