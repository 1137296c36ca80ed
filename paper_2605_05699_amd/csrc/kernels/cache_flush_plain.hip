// A cache's flush: the plain form of the write path, alone (the record by the way of srft_flush_staged) and with the plain form of the
// read path behind it.
#include "../cache_flush.h"

namespace {
template <int D, int S, int GM, int BITS>
flush_kernels_t kernels(bool staged) {
    constexpr int NT = 2 * D / S, KS = GM == kGroup16 ? 1 : 2;
    const auto alone = [&](auto lanes, auto lds) { return staged ? lds : lanes; };
    const auto write = alone(srft_cache_flush_kernel<D, NT, srft_flush_write_plain<D, S, GM, BITS, srft_flush_staged(D, 1)>, srft_flush_read_later>,
                             srft_cache_flush_kernel<D, NT, srft_flush_write_plain<D, S, GM, BITS, srft_flush_staged(D, 1LL << 40)>, srft_flush_read_later>);
    if constexpr (D <= 128)
        return {write, srft_cache_flush_kernel<D, NT, srft_flush_write_plain<D, S, GM, BITS, false>, srft_flush_read_plain<D, S, KS, BITS>>};
    else
        return {write, nullptr};
}
template <int D>
flush_kernels_t pick(int bits, int gm, bool staged) {
    constexpr int S = D == 64 ? 2 : 1;
    if (bits == 8)
        return gm == kGroup16 ? kernels<D, S, kGroup16, 8>(staged) : gm == kGroupWide ? kernels<D, S, kGroupWide, 8>(staged) : kernels<D, S, kGroup32, 8>(staged);
    return gm == kGroup16 ? kernels<D, S, kGroup16, 4>(staged) : gm == kGroupWide ? kernels<D, S, kGroupWide, 4>(staged) : kernels<D, S, kGroup32, 4>(staged);
}
flush_kernels_t dispatch(int d, int bits, int gm, bool staged) {
    SRFT_DISPATCH_D(d, pick, bits, gm, staged)
}
}  // namespace

flush_kernels_t srft_pick_cache_flush_plain(int d, int bits, int gm, bool staged) { return dispatch(d, bits, gm, staged); }
