// quantize_tiles.h -- write path, plain form: the kernel template and its per-plan and batched kernels.
#ifndef SRFT_QUANTIZE_TILES_H
#define SRFT_QUANTIZE_TILES_H
#include "device_util.h"

// ------------------------------------------------------------------------------------------
// write path
// ------------------------------------------------------------------------------------------
// wfrag : [D/32 slabs][D/16 k-steps][hi, lo][64 lanes] 16-byte A-operand fragments of W
// x     : [n_vec][D/8] 16-byte units of fp16 input
// S     : slabs (= quantization groups) per wavefront; the workgroup has D / (32 S) wavefronts.  With S = 2 (d = 64) every
//         B fragment read from LDS feeds four MFMAs instead of two; the price is a 2 x larger register-resident slab.
// OUT   : kOutCodes: the quantizer.  kOutRaw: store the fp32 coefficients w instead (srft_kv_forward_f32).
//         kOutAmax: no per-vector output; every lane keeps the running maximum of |w| of its 16 channels over the
//         tiles it sees, the lanes' maxima meet in LDS once at the end and one atomic max per channel and workgroup
//         goes to wout, read as float[d] (srft_kv_channel_absmax: the statistic lambda is calibrated from, Sec. 7.1).
// GM    : group mode.  kGroup32: one scale per slab (g = 32, the deployed format).  kGroup16: one scale per
//         lane (g = 16; a lane's 16 outputs are one group, no cross-lane step).  kGroupWide: g = 32 * gw with
//         gw >= 2 slabs per group, up to the per-token case g = d; the slab maxima meet in LDS, which costs
//         two more barriers per tile.
// The work of one workgroup: tiles t0, t0 + stride, ... of one plan's n_vec vectors (t0 < number of tiles).
// BITS  : 4 (two nibbles per byte) or 8 (one byte per value, scale = abs-max / 127; Sec. 3.2 steps 3-4)
// STAGED: the record goes through LDS and is written through to memory (srft_write_staged).
// SUB   : teams of G / S wavefronts per workgroup (kOutAmax), as in srft_quantize_fold_tiles
template <int D, int S, int OUT, int GM, int BITS, bool STAGED, int SUB = 1, class ROWS = srft_rows_dense>
__device__ __forceinline__ void
srft_quantize_tiles(const uint4* __restrict__ wfrag, const uint4* __restrict__ x, long long n_vec,
                    uint2* __restrict__ codes, float* __restrict__ scales, float4* __restrict__ wout,
                    float unscale, float scale_mul, int gw, const int first_tile, const int stride, const ROWS& rows = ROWS()) {
    static_assert(SUB == 1 || OUT == kOutAmax, "records are written by one team");
    constexpr int G = D / 32;            // quantization groups per vector = slabs of the matrix
    constexpr int T = D / 16;            // MFMA k-steps
    constexpr int U = D / 8;             // 16-byte units per input row
    constexpr int ROW = U + 1;           // padded LDS row (odd number of units: conflict-free b128 reads)
    constexpr int NT = 64 * G / S;       // threads per workgroup
    constexpr int PER = 2 * S;           // 16-byte units each thread moves per tile (32 * U = PER * NT)
    constexpr int TB = (T < 8) ? T : 8;  // B fragments read from LDS ahead of their MFMAs
    static_assert(G % S == 0, "slabs per wavefront must divide the number of groups");
    __shared__ uint4 lds_of[SUB][2][kTileVecs * ROW];
    __shared__ float gmax[GM == kGroupWide ? kTileVecs * G : 1];     // per (vector, slab) abs-max
    // the record of a finished tile, stored one stage later as whole rows (STAGED)
    constexpr bool STAGE = OUT == kOutCodes && STAGED;
    constexpr int CU8 = D * BITS / 64, CROW = CU8 + 1;       // 8-byte units per code row; padded
    constexpr int SMAX = GM == kGroup16 ? 2 * G : G;         // most scales of a vector
    __shared__ uint2 cstage[STAGE ? 2 : 1][STAGE ? kTileVecs * CROW : 1];
    __shared__ float sstage[STAGE ? 2 : 1][STAGE ? kTileVecs * SMAX : 1];

    const int team = SUB > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NT) : 0, t0 = first_tile + team;
    auto& lds = lds_of[team];
    const int tid = threadIdx.x - team * NT, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    // tile indices are 32-bit (the host bounds n_vec), so that the uniform index arithmetic stays scalar
    const int n_tiles = (int)((n_vec + kTileVecs - 1) / kTileVecs);
    const int last_lim = (int)(n_vec - 1 - (long long)(n_tiles - 1) * kTileVecs);   // last valid row of the last tile

    half8 ahi[S][T], alo[S][T];

    // The PER prefetched units of one tile live in separately named registers (PER = 2 uses a and b only).
    // Addresses are a uniform tile base (scalar registers) plus a 32-bit per-lane offset; rows past the end
    // alias to the last row through `lim`, the index of the last valid row of the tile (uniform).
    auto fetch1 = [&](uint4& v, int i, const uint4* tile_base, int lim, int tile) __attribute__((always_inline)) {
        const int u = tid + i * NT, r = u / U, c = u % U;
        if constexpr (std::is_same_v<ROWS, srft_rows_dense>) v = tile_base[(unsigned)(min(r, lim) * U + c)];
        else v = rows.template row<U>(tile * kTileVecs + min(r, lim))[c];
    };
    auto fetch = [&](uint4& a, uint4& b, uint4& c, uint4& d, int tile) __attribute__((always_inline)) {
        if (tile > n_tiles - 1) tile = n_tiles - 1;          // prefetch past the end re-reads the last tile
        const long long row0 = (long long)tile * kTileVecs;
        const int lim = (tile == n_tiles - 1) ? last_lim : kTileVecs - 1;
        const uint4* tile_base = x + row0 * U;
        fetch1(a, 0, tile_base, lim, tile);
        fetch1(b, 1, tile_base, lim, tile);
        if constexpr (PER > 2) { fetch1(c, 2, tile_base, lim, tile); fetch1(d, 3, tile_base, lim, tile); }
    };
    auto put1 = [&](int buf, const uint4& v, int i) __attribute__((always_inline)) {
        const int u = tid + i * NT, r = u / U, c = u % U;
        lds[buf][r * ROW + c] = v;
    };
    auto to_lds = [&](int buf, const uint4& a, const uint4& b, const uint4& c, const uint4& d) __attribute__((always_inline)) {
        put1(buf, a, 0);
        put1(buf, b, 1);
        if constexpr (PER > 2) { put1(buf, c, 2); put1(buf, d, 3); }
    };
    float cmax[OUT == kOutAmax ? S : 1][16] = {};            // running per-channel maxima (kOutAmax)
    using Acc = Accs<S>;
    auto contract = [&](int b, Acc& accs) __attribute__((always_inline)) {
        const uint4* rowp = &lds[b][col * ROW + half];
        each_acc(accs, [&](floatx16& acc, int) __attribute__((always_inline)) { acc = floatx16{0}; });
#pragma unroll
        for (int t0 = 0; t0 < T; t0 += TB) {
            half8 bf[TB];
#pragma unroll
            for (int t = 0; t < TB; ++t)
                if (t0 + t < T) bf[t] = __builtin_bit_cast(half8, rowp[2 * (t0 + t)]);
#pragma unroll
            for (int t = 0; t < TB; ++t)
                if (t0 + t < T) {
                    each_acc(accs, [&](floatx16& acc, int s) __attribute__((always_inline)) {
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ahi[s][t0 + t], bf[t], acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(alo[s][t0 + t], bf[t], acc, 0, 0, 0);
                    });
                }
        }
    };
    [[maybe_unused]] const int ns = GM == kGroupWide ? G / gw : SMAX;
    // vector-ALU tail of one tile: per-group abs-max, scale, int4 codes, into staging buffer b or to memory
    auto finish = [&](Acc& accs, int tile, [[maybe_unused]] const int b) __attribute__((always_inline)) {
        const long long row0 = (long long)tile * kTileVecs;
        const int lim = (tile == n_tiles - 1) ? last_lim : kTileVecs - 1;     // uniform
        const int c = min(col, lim);                                      // alias rows past the end
        if constexpr (OUT == kOutAmax) {
            // rows past the end repeat the last row, which changes no maximum
            each_acc(accs, [&](floatx16& acc, int s) __attribute__((always_inline)) {
#pragma unroll
                for (int v = 0; v < 16; ++v) cmax[s][v] = fmaxf(cmax[s][v], fabsf(acc[v]));
            });
        } else if constexpr (OUT == kOutRaw) {
            each_acc(accs, [&](floatx16& acc, int s) __attribute__((always_inline)) {
                const int slab = wave * S + s;
                float4* o = wout + (row0 * D) / 4 + (unsigned)((c * D + 32 * slab + 16 * half) / 4);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    o[i] = make_float4(acc[4 * i] * unscale, acc[4 * i + 1] * unscale,
                                       acc[4 * i + 2] * unscale, acc[4 * i + 3] * unscale);
            });
        } else {
            float mm[S];
            each_acc(accs, [&](floatx16& acc, int s) __attribute__((always_inline)) {
                float m = fmaxf(fabsf(acc[0]), fabsf(acc[1]));
#pragma unroll
                for (int v = 2; v < 16; ++v) m = fmaxf(m, fabsf(acc[v]));
                if constexpr (GM != kGroup16) m = other_half_max(m);
                mm[s] = m;
            });
            if constexpr (GM == kGroupWide) {
                __syncthreads();                             // the previous tile's maxima have been read
#pragma unroll
                for (int s = 0; s < S; ++s) gmax[col * G + wave * S + s] = mm[s];
                __syncthreads();
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const int first = (wave * S + s) / gw * gw;
                    float m = gmax[col * G + first];
                    for (int i = 1; i < gw; ++i) m = fmaxf(m, gmax[col * G + first + i]);
                    mm[s] = m;
                }
            }
            each_acc(accs, [&](floatx16& acc, int s) __attribute__((always_inline)) {
                const int slab = wave * S + s;
                float scale = mm[s] * scale_mul;             // scale_mul = fl(2^-e / 7): abs-max / 7
                float inv = unscale * __builtin_amdgcn_rcpf(scale);
                if (!(scale >= kMinScale)) { scale = 0.0f; inv = 0.0f; }
                if constexpr (!STAGE) {
                    if constexpr (BITS == 8) {   // 16 bytes per lane; a row is D / 16 such units
                        const uint4 packed = make_uint4(pack4_bytes(acc, 0, inv), pack4_bytes(acc, 4, inv),
                                                        pack4_bytes(acc, 8, inv), pack4_bytes(acc, 12, inv));
                        (reinterpret_cast<uint4*>(codes) + row0 * (D / 16))[(unsigned)(c * (D / 16) + 2 * slab + half)] = packed;
                    } else {
                        uint2 packed;
                        packed.x = pack8(acc, 0, inv);
                        packed.y = pack8(acc, 8, inv);
                        (codes + row0 * (D / 16))[(unsigned)(c * (D / 16) + 2 * slab + half)] = packed;
                    }
                    // lanes that hold the same group store the same value to the same place
                    if constexpr (GM == kGroup16) (scales + row0 * (2 * G))[(unsigned)(c * (2 * G) + 2 * slab + half)] = scale;
                    else if constexpr (GM == kGroup32) (scales + row0 * G)[(unsigned)(c * G + slab)] = scale;
                    else (scales + row0 * (G / gw))[(unsigned)(c * (G / gw) + slab / gw)] = scale;
                    return;
                }
                uint2* const crow = &cstage[b][col * CROW + (2 * slab + half) * (BITS / 4)];
                if constexpr (BITS == 8) {
                    crow[0] = make_uint2(pack4_bytes(acc, 0, inv), pack4_bytes(acc, 4, inv));
                    crow[1] = make_uint2(pack4_bytes(acc, 8, inv), pack4_bytes(acc, 12, inv));
                } else {
                    crow[0] = make_uint2(pack8(acc, 0, inv), pack8(acc, 8, inv));
                }
                sstage[b][col * ns + (GM == kGroup16 ? 2 * slab + half : GM == kGroup32 ? slab : slab / gw)] = scale;
            });
        }
    };

    // staged record of `tile` -> global memory, whole rows next to each other (rows past the end alias to the last row; lanes
    // without a scale store behind the end of the buffer, that is nowhere)
    auto flush = [&](int b, int tile) __attribute__((always_inline)) {
        if constexpr (STAGE) {
            const long long row0 = (long long)tile * kTileVecs;
            const int lim = (tile == n_tiles - 1) ? last_lim : kTileVecs - 1;
            constexpr int WIDTH = BITS * S >= 8 ? 2 : 1, ROWS_OF = CU8 / WIDTH, PIECES = kTileVecs * ROWS_OF;    // 8-byte units a piece
            static_assert(PIECES % NT == 0, "as many pieces for every thread");
            uint2* const cbase = codes + row0 * CU8;
#pragma unroll
            for (int i = 0; i < PIECES / NT; ++i) {
                const int u = tid + i * NT, r = u / ROWS_OF, p = u % ROWS_OF;
                const uint2* const from = &cstage[b][r * CROW + WIDTH * p];
                const unsigned at = __umul24(min(r, lim), CU8) + WIDTH * p;
                if constexpr (WIDTH == 2) stream_store<kStoreThroughOnce>(cbase, at, make_uint4(from[0].x, from[0].y, from[1].x, from[1].y));
                else stream_store<kStoreThroughOnce>(cbase, at, from[0]);
            }
#pragma unroll
            for (int i = 0; i < (kTileVecs * SMAX + NT - 1) / NT; ++i) {
                const int e = tid + i * NT;
                const int r = GM == kGroupWide ? e / ns : e / SMAX, j = GM == kGroupWide ? e % ns : e % SMAX;
                const bool mine = e < kTileVecs * ns;
                stream_store<kStoreThrough>(scales + row0 * ns, (unsigned)(min(r, lim) * ns + j), sstage[b][mine ? e : 0], mine);
            }
        }
    };

    const int m = (n_tiles - 1 - first_tile) / stride + 1;   // tiles of a team: t0, t0 + stride, ...
    uint4 pa0, pa1, pa2, pa3, pb0, pb1, pb2, pb3;
    Acc acc_a, acc_b;
    fetch(pa0, pa1, pa2, pa3, t0);
    // The first tile is asked for ahead of the matrix (it comes from farther away, and does not wait for the plan's entry), the
    // second one behind it: the first tile goes to LDS while the matrix is on its way.
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            ahi[s][t] = __builtin_bit_cast(half8, wfrag[(((wave * S + s) * T + t) * 2 + 0) * 64 + lane]);
            alo[s][t] = __builtin_bit_cast(half8, wfrag[(((wave * S + s) * T + t) * 2 + 1) * 64 + lane]);
        }
    __builtin_amdgcn_sched_barrier(0);
    fetch(pb0, pb1, pb2, pb3, t0 + stride);
    to_lds(0, pa0, pa1, pa2, pa3);
    hold_in_registers(ahi, alo);                 // the matrix slab has arrived before the pipeline starts
    fetch(pa0, pa1, pa2, pa3, t0 + 2 * stride);
    // stage 0
    __syncthreads();
    contract(0, acc_a);
    to_lds(1, pb0, pb1, pb2, pb3);
    fetch(pb0, pb1, pb2, pb3, t0 + 3 * stride);
    int k = 1;
    for (; k + 1 < m; k += 2) {
        const int tk = t0 + k * stride;
        __syncthreads();                         // stage k (odd)
        rotate_priority(k + team);
        if constexpr (STAGE)
            if (k >= 2) flush(1, tk - 2 * stride);
        contract(1, acc_b);
        finish(acc_a, tk - stride, 0);
        to_lds(0, pa0, pa1, pa2, pa3);
        fetch(pa0, pa1, pa2, pa3, tk + 3 * stride);
        __syncthreads();                         // stage k + 1 (even)
        rotate_priority(k + 1 + team);
        flush(0, tk - stride);
        contract(0, acc_a);
        finish(acc_b, tk, 1);
        to_lds(1, pb0, pb1, pb2, pb3);
        fetch(pb0, pb1, pb2, pb3, tk + 4 * stride);
    }
    if (k < m) {                                 // one more odd stage
        const int tk = t0 + k * stride;
        __syncthreads();
        if constexpr (STAGE)
            if (k >= 2) flush(1, tk - 2 * stride);
        contract(1, acc_b);
        finish(acc_a, tk - stride, 0);
        if constexpr (STAGE) __syncthreads();    // (staging buffer 1 has been read, buffer 0 is full)
        flush(0, tk - stride);
        finish(acc_b, tk, 1);
        if constexpr (STAGE) __syncthreads();
        flush(1, tk);
    } else {
        const int tl = t0 + (k - 1) * stride;
        if constexpr (STAGE) {
            __syncthreads();
            if (k >= 2) flush(1, tl - stride);
        }
        finish(acc_a, tl, 0);
        if constexpr (STAGE) __syncthreads();
        flush(0, tl);
    }
    if constexpr (OUT == kOutAmax) {
        // lanes of one half hold the same 16 channels for 32 different vectors: they meet in LDS (the tile buffers, which
        // no wavefront reads any more), then one atomic per channel
        static_assert(sizeof(lds) >= sizeof(float) * kTileVecs * kAmaxRow<D> && NT >= D, "room and a thread per channel");
        __syncthreads();
        float* part = reinterpret_cast<float*>(&lds[0][0]);
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int v = 0; v < 16; ++v) part[col * kAmaxRow<D> + 32 * (wave * S + s) + 16 * half + v] = cmax[s][v];
        publish_amax<D, SUB>(reinterpret_cast<float*>(&lds_of[0][0][0]), sizeof(lds_of[0]) / sizeof(float), reinterpret_cast<unsigned int*>(wout), unscale);
    }
}

// Wavefronts per SIMD that the registers are to leave room for.  With the record's way through LDS the compiler takes 10 to 15
// registers more: at d = 128 3 past the step to one wavefront less, which it finds again when asked (at d = 96 9 past it: asked, it
// spills 6 to 20).
template <int D, bool STAGED> constexpr int kQuantizeWaves = STAGED && D == 128 ? 3 : 1;
template <int D, int S, int OUT, int GM, int BITS, bool STAGED, int SUB = 1>
__global__ void __launch_bounds__(2 * D / S * SUB, (kQuantizeWaves<D, STAGED>))
srft_quantize_kernel(const uint4* __restrict__ wfrag, const uint4* __restrict__ x, long long n_vec,
                     uint2* __restrict__ codes, float* __restrict__ scales, float4* __restrict__ wout,
                     float unscale, float scale_mul, int gw) {
    srft_quantize_tiles<D, S, OUT, GM, BITS, STAGED, SUB>(wfrag, x, n_vec, codes, scales, wout, unscale, scale_mul, gw, blockIdx.x * SUB,
                                       gridDim.x * SUB);     // no workgroup without a tile
}

// Several plans in one launch (see srft_batch).
template <int D, int S, int GM, int BITS, bool STAGED, int N>
__global__ void __launch_bounds__(2 * D / S, (kQuantizeWaves<D, STAGED>))
srft_quantize_batched_kernel(const srft_batch<N> a, int gw) {
    const srft_work s = srft_work_of_block<true>(a);
    srft_quantize_tiles<D, S, kOutCodes, GM, BITS, STAGED>(s.frag, (const uint4*)s.in, s.n_vec, (uint2*)s.out, s.scales,
                                         nullptr, s.unscale, s.unscale / (BITS == 8 ? 127.0f : 7.0f), gw, s.place, s.blocks);
}

#endif  // SRFT_QUANTIZE_TILES_H
