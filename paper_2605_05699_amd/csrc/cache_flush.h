// cache_flush.h -- an append to a cache that fills pages: the tokens of these pages are quantized from where the caller has them
// (and from the view, where the window holds the first ones), those behind the last full page are copied into the window, and
// the pages are decoded into the view, in the same launch or in one behind it.
//
// A flush during decoding is one tile of 32 vectors per plan, and the copy into the window, the quantizer and the read path were
// a launch each, all latency (2.0-2.5 us of the host each; 2.4 + 3.9 + 4.1 us on the device, with the gaps).  Here a
// workgroup takes its tiles through both paths, one after the other, and reads back its own records, which the caches near it
// still hold.  A prompt is no longer copied into the view, to be read from there and overwritten.  The two halves' registers are
// one allocation, their LDS adds up (60 KB at d = 128, 148 KB at d = 256), so from a few tiles per workgroup on the read path,
// which could have more workgroups, is a launch of its own (srft_flush_whole_tiles).  Device time of one append over 56 plans, us,
// copy + quantizer + read path -> write half, read path apart / whole:
//   d = 128   2 x 16 tokens 8.95 -> 7.2 / 6.0   2 x 256 16.6 -> 10.7 / 8.7    2 x 1000 33.5 -> 22.6 / 23.2   8 x 1000 103 -> 63 / 74
//   d = 256   2 x 16 10.9 -> 8.7 / 7.4          2 x 320 27.7 -> 19.7 / 19.9   2 x 500 36.4 -> 24.9 / 29.2    8 x 3000 644 -> 389 / 509
//     g = 16  2 x 128 20.0 -> 12.4 / 11.2       2 x 256 29.4 -> 16.8 / 17.8   2 x 1000 84.5 -> 43.3 / 56.0
//   d = 96    2 x 16 8.2 -> 6.4 / 4.6           2 x 500 19.6 -> 13.3 / 12.0   3 x 1000 41.3 -> 26.0 / 24.2   8 x 3000 261 -> 145 / 147
//   d = 64    2 x 16 7.9 -> 6.2 / 4.7           3 x 1000 26.9 -> 17.6 / 17.0  8 x 1000 56.2 -> 32.2 / 33.9   8 x 3000 143 -> 90 / 92
//   d = 128, g = 16   2 x 128 12.8 -> 8.7 / 7.1    2 x 256 17.6 -> 12.2 / 12.9    2 x 500 24.7 -> 17.4 / 19.7
//   d = 32    2 x 16 6.85 -> 5.0 / 3.6          3 x 1000 15.4 -> 10.1 / 9.2   8 x 1000 29.5 -> 17.9 / 19.7   8 x 3000 76.4 -> 40.3 / 47.9
#ifndef SRFT_CACHE_FLUSH_H
#define SRFT_CACHE_FLUSH_H
#include "dequantize_fold4_tiles.h"
#include "dequantize_tiles.h"
#include "quantize_fold4_tiles.h"
#include "quantize_fold_tiles.h"
#include "quantize_tiles.h"

// The two halves of a plan's forms, for workgroups of one size.
template <int D, int S, int GM, int BITS, bool STAGED>
struct srft_flush_write_plain {
    static __device__ __forceinline__ void run(const uint4* frag, float unscale, const srft_flush& a, uint2* codes, float* scales,
                                               const srft_rows_paged& rows, int place, int blocks) {
        srft_quantize_tiles<D, S, kOutCodes, GM, BITS, STAGED>(frag, nullptr, a.n_vec, codes, scales, nullptr, unscale,
                                                       unscale / (BITS == 8 ? 127.0f : 7.0f), a.gw, place, blocks, rows);
    }
};
template <int D, int BITS, bool WIDE>
struct srft_flush_write_fold {
    static __device__ __forceinline__ void run(const uint4* frag, float unscale, const srft_flush& a, uint2* codes, float* scales,
                                               const srft_rows_paged& rows, int place, int blocks) {
        srft_quantize_fold_tiles<D, BITS, WIDE>(frag, nullptr, a.n_vec, codes, scales, unscale, unscale / (BITS == 8 ? 127.0f : 7.0f),
                                                a.gw, place, blocks, (a.n_vec + kTileVecs - 1) / kTileVecs, nullptr, rows);
    }
};
template <int BITS, int GM>
struct srft_flush_write_fold4 {
    static __device__ __forceinline__ void run(const uint4* frag, float, const srft_flush& a, uint2* codes, float* scales,
                                               const srft_rows_paged& rows, int place, int blocks) {
        srft_quantize_fold4_tiles<BITS, GM>(frag, nullptr, a.n_vec, codes, scales, 1.0f / (BITS == 8 ? 127.0f : 7.0f), place, blocks,
                                            (a.n_vec + kTileVecs - 1) / kTileVecs, nullptr, rows);
    }
};
template <int D, int S, int KS, int BITS>
struct srft_flush_read_plain {
    static __device__ __forceinline__ void run(const uint4* frag, float unscale, const srft_flush& a, const uint2* codes,
                                               const float* scales, uint4* view, int place, int blocks) {
        srft_dequantize_tiles<D, S, KS, false, BITS>(frag, codes, scales, a.n_vec, view, unscale, a.gw, place, blocks,
                                                     (a.n_vec + kTileVecs - 1) / kTileVecs);
    }
};
template <int D, int BITS, bool FINE = false>
struct srft_flush_read_fold4 {
    static __device__ __forceinline__ void run(const uint4* frag, float unscale, const srft_flush& a, const uint2* codes,
                                               const float* scales, uint4* view, int place, int blocks) {
        srft_dequantize_fold4_tiles<D, BITS, FINE>(frag, codes, scales, a.n_vec, view, unscale, a.gw, place, blocks,
                                             (a.n_vec + kTileVecs - 1) / kTileVecs);
    }
};

struct srft_flush_read_later {};             // (a launch of its own)

template <int D, int NT, class WRITE, class READ>
__global__ void __launch_bounds__(NT, NT == D && D >= 128 ? 2 : 1)
srft_cache_flush_kernel(const srft_flush a) {
    constexpr int U = D / 8;
    const int block = srft_block_by_die();
    const int i = srft_even_segment(block, a.shape), start = srft_even_start(i, a.shape);
    const int blocks = srft_even_start(i + 1, a.shape) - start, place = block - start;
    const srft_plan_entry* e = reinterpret_cast<const srft_plan_entry*>(reinterpret_cast<const char*>(a.plan) + i * a.plan_step);
    uint4* const view = reinterpret_cast<uint4*>(a.view + i * a.view_step);
    uint2* const codes = reinterpret_cast<uint2*>(a.codes + i * a.codes_step);
    float* const scales = reinterpret_cast<float*>(a.scales + i * a.scales_step);
    const uint4* const fresh = reinterpret_cast<const uint4*>(a.fresh + i * a.fresh_step);
    const auto table = [&](int path) { return (const uint4*)(const __attribute__((address_space(1))) uint4*)e->table[path]; };
    WRITE::run(table(0), e->unscale[0], a, codes, scales,
               {fresh, view, a.page_rows, a.R, a.held, a.t_all, a.page_magic, a.slot_magic}, place, blocks);
    // the tokens behind the last full page
    const int per = a.tail * U;
    for (int k = place * NT + threadIdx.x; k < a.page_rows / a.R * per; k += blocks * NT) {
        const int seq = k / per, u = k % per;
        view[(unsigned)((a.n_vec + seq * a.R) * U + u)] = fresh[(unsigned)((seq * a.t_all + a.t_all - a.tail) * U + u)];
    }
    if constexpr (!std::is_same_v<READ, srft_flush_read_later>) {
        __syncthreads();                         // the records of this workgroup's tiles are written, the rows they came from read
        READ::run(table(1), e->unscale[1], a, codes, scales, view, place, blocks);
    }
}

#endif  // SRFT_CACHE_FLUSH_H
