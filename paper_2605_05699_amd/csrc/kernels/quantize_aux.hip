// Write path, plain form, outputs other than codes: the raw coefficients (srft_kv_forward_f32) and the
// per-channel abs-max statistic (srft_kv_channel_absmax).
#include "../quantize_tiles.h"

namespace {
template <int D, int S>
quantize_kernel_t by_output(int out, int teams) {
    if (out == kOutRaw) return srft_quantize_kernel<D, S, kOutRaw, kGroup32, 4, false>;
    if (out != kOutAmax) return nullptr;
    constexpr int MANY = D == 32 ? 8 : D == 64 || D == 96 ? 4 : D == 128 ? 2 : 1;
    return teams == 1      ? srft_quantize_kernel<D, S, kOutAmax, kGroup32, 4, false, 1>
           : teams == MANY ? srft_quantize_kernel<D, S, kOutAmax, kGroup32, 4, false, MANY>
                           : nullptr;
}
template <int D>
quantize_kernel_t pick(int slabs, int out, int teams) {
    if constexpr (D == 64) {
        if (slabs == 2) return by_output<D, 2>(out, teams);
    }
    return by_output<D, 1>(out, teams);
}
}  // namespace

quantize_kernel_t srft_pick_quantize_aux(int d, int slabs, int out, int teams) { SRFT_DISPATCH_D(d, pick, slabs, out, teams) }
