// Scores of queries against the stored keys, in the rotated domain.
//
// <q, k_t> with k_t = s * Q^T (code * scale / lambda) equals <q', code * scale> with q' = Q (s * q) / lambda:
// the transform is orthogonal, so the keys never have to be reconstructed; the kernel reads the 4-bit record
// only (d/2 + 4 d/g bytes per key instead of the 2d of a dequantized prefix) and writes n_q floats per key.
//
// One launch.  Every workgroup forms q' (rotated_queries.h); a wavefront walks over tiles of 64 or 32 keys.  Keys are the
// rows and queries the columns of v_mfma_f32_16x16x32_f16: the codes of a key go from global memory into the A operand with
// a transpose over the wavefront's quarters and never through LDS, and a lane ends up with 4 consecutive keys of ITS query
// per block of 16 -- one 16-byte store, 64 bytes next to each other per query (with more than 8 queries whole lines, by way
// of LDS).  With more than 16 queries both blocks of 16 take the same decoded keys.  At many keys it is bound by memory, at
// few by the chain of one launch.  Measured, us, against a launch for q' and a scan by one-wavefront workgroups that decoded
// the codes into LDS (and wrote a query's keys with 4-byte stores): d = 128, 8 queries: 20,000 keys 13.1 -> 7.9, 1,000,000
// keys 30.0 -> 21.6 (112 MB: 5.2 TB/s); 32 queries, 300,000 keys 24.6 -> 15.2; d = 64, 8 queries, 1,000,000 keys 20.6 ->
// 14.8; d = 256 59.4 -> 36.4.
#include "../rotated_queries.h"

namespace {

constexpr int kWaves = 8;                        // wavefronts per workgroup
// keys per tile (one wavefront): 32 where a tile of 64 would leave up to 200 registers in scratch
template <int D, int RB> constexpr int kTileKeys = D * RB > 256 || D == 256 ? 32 : 64;

// D: head dimension.  RB: blocks of 16 queries.  WIDE: groups of gw > 1 runs of 32 channels share a scale.
// STAGE: scores go out by way of LDS (more than 8 queries).  Many queries are mostly stores, and one from the registers writes
// 64 bytes each of 16 queries; from LDS it writes whole lines of a few.  us, d = 64, 32 queries, 2,000,000 keys 86 -> 74,
// 16 queries, 1,000,000 keys 27.0 -> 21.5; d = 128, 32 queries 49 -> 45.  With half-empty blocks it is slower at 300,000 keys
// (8 queries, d = 64 7.4 -> 7.6) and with one query everywhere (1,000,000 keys 10.4 -> 11.0).
// codes [n_keys][D / 2] bytes, scales [n_keys][D / 32 / gw], out [n_q][n_keys]
template <int D, int RB, bool WIDE, bool STAGE, bool THROUGH>
__global__ void __launch_bounds__(64 * kWaves, 2)
srft_scores_kernel(const uint4* __restrict__ q, int n_q, const uint4* __restrict__ q_table, int hadamard,
                   const uint8_t* __restrict__ codes, const float* __restrict__ scales, int gw,
                   long long n_keys, float* __restrict__ out) {
    constexpr int G = D / 32, QUADS = G / 4, REST = G % 4;   // a row of codes: QUADS x 64 bytes, then REST x 16 bytes
    constexpr int ROW = D / 2, W = kWaves, KEYS = kTileKeys<D, RB>, BK = KEYS / 16;
    constexpr int SCRATCH = srft_query_scratch_bytes<D, RB>(), TILES = W * G * KEYS * 4;
    __shared__ __align__(16) unsigned char lds[SCRATCH > TILES ? SCRATCH : TILES];
    __shared__ uint4 qs[RB * G * 2 * 64];
    constexpr int SROW = KEYS + 4;                           // padded
    __shared__ __align__(16) float staged[STAGE ? W * 16 * SROW : 4];        // [wavefront][query of a block][key]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, a = lane >> 4;                // query (or key of a block of 16), quarter
    float* const ks = reinterpret_cast<float*>(lds) + wave * G * KEYS;      // this wavefront's scales, [group][key]
    const long long n_tiles = (n_keys + KEYS - 1) / KEYS, stride = (long long)gridDim.x * W;
    const long long first = (long long)wave * gridDim.x + blockIdx.x;

    uint4 pk[BK][QUADS ? QUADS : 1];
    static_assert(REST == 0 || REST == 2, "d is a multiple of 64");
    uint2 pr[BK];
    floatx4 ps[(G + 3) / 4];
    // keys past the end alias to the last one; all = false: every lane reads the tile's first key (there is no next tile)
    auto fetch = [&](long long tile, bool all) __attribute__((always_inline)) {
        const long long t0 = tile * KEYS;
        const int lim = all ? (int)min((long long)(KEYS - 1), n_keys - 1 - t0) : 0;
        const uint8_t* kb = codes + t0 * ROW;
#pragma unroll
        for (int b = 0; b < BK; ++b) {
            const unsigned row = (unsigned)min(16 * b + l16, lim) * ROW;
#pragma unroll
            for (int s = 0; s < QUADS; ++s) pk[b][s] = *reinterpret_cast<const uint4*>(kb + (row + 64 * s + 16 * a));
            if constexpr (REST > 0) pr[b] = *reinterpret_cast<const uint2*>(kb + (row + 64 * QUADS + 8 * a));
        }
        const int rl = min(lane & (KEYS - 1), lim);
        if constexpr (WIDE) {
            const int ns = G / gw;
#pragma unroll
            for (int j = 0; j < G; ++j) ps[j / 4][j % 4] = (scales + t0 * ns)[(unsigned)(rl * ns + j / gw)];
        } else {
            const float* row = scales + t0 * G + (unsigned)(rl * G);
#pragma unroll
            for (int j = 0; j + 4 <= G; j += 4) ps[j / 4] = *reinterpret_cast<const floatx4u*>(row + j);
#pragma unroll
            for (int j = G / 4 * 4; j < G; ++j) ps[j / 4][j % 4] = row[j];
        }
    };
    srft_query_operands<D, W, RB>(q, n_q, 0, q_table, hadamard, 1.0f, lds, qs, [&]() __attribute__((always_inline)) {
        fetch(min(first, n_tiles - 1), first < n_tiles);
    });

    for (long long tile = first; tile < n_tiles; tile += stride) {           // uniform per wavefront; no barrier inside
        const bool more = tile + stride < n_tiles;
        const long long t0 = tile * KEYS;
#pragma unroll
        for (int j = 0; j < G; ++j) ks[j * KEYS + (lane & (KEYS - 1))] = ps[j / 4][j % 4];
        uint32_t kd[BK][G];                                  // dword of unit `a` of every group
#pragma unroll
        for (int b = 0; b < BK; ++b) {
#pragma unroll
            for (int s = 0; s < QUADS; ++s) {
                const uint4 r = srft_quad_transpose(pk[b][s]);
                kd[b][4 * s] = r.x;
                kd[b][4 * s + 1] = r.y;
                kd[b][4 * s + 2] = r.z;
                kd[b][4 * s + 3] = r.w;
            }
            if constexpr (REST > 0) {
                const uint2 r = srft_pair_transpose(pr[b]);
                kd[b][4 * QUADS] = r.x;
                kd[b][4 * QUADS + 1] = r.y;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");               // LDS of one wavefront: in program order
        __builtin_amdgcn_sched_barrier(0);
        fetch(more ? tile + stride : tile, more);            // (not under a branch: see kernels/decode_attention.hip)
        // (the queries' operands are the same for every tile; more than 32 registers of them are read from LDS again)
        int at = lane;
        if constexpr (RB * G > 4) asm volatile("" : "+v"(at));
        floatx4 w[RB][BK];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            half8 qh[RB], ql[RB];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                qh[rb] = __builtin_bit_cast(half8, qs[((rb * G + j) * 2 + 0) * 64 + at]);
                ql[rb] = __builtin_bit_cast(half8, qs[((rb * G + j) * 2 + 1) * 64 + at]);
            }
#pragma unroll
            for (int b = 0; b < BK; ++b) {
                const half8 kf = __builtin_bit_cast(half8, decode8(kd[b][j]));
                const floatx4 sc = *reinterpret_cast<const floatx4*>(&ks[j * KEYS + 16 * b + 4 * a]);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    floatx4 s = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qh[rb], floatx4{0, 0, 0, 0}, 0, 0, 0);
                    s = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, ql[rb], s, 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[rb][b][i] = j == 0 ? s[i] * sc[i] : fmaf(s[i], sc[i], w[rb][b][i]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);               // one group's operands at a time (registers)
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int mine = (int)min((long long)KEYS, n_keys - t0) - 4 * a;    // keys of the tile from this quarter's first on
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int query = 16 * rb + l16;
            float* const row = out + (long long)min(query, n_q - 1) * n_keys + t0 + 4 * a;
            if (STAGE && t0 + KEYS <= n_keys) {              // uniform
                float* const st = staged + wave * 16 * SROW;
#pragma unroll
                for (int b = 0; b < BK; ++b) *reinterpret_cast<floatx4*>(&st[l16 * SROW + 16 * b + 4 * a]) = w[rb][b];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                constexpr int L = KEYS / 4, R = 64 / L;      // lanes per query, queries per store
#pragma unroll
                for (int i = 0; i < 16; i += R) {
                    const int mine = i + lane / L, c = 4 * (lane % L);
                    const floatx4 v = *reinterpret_cast<const floatx4*>(&st[mine * SROW + c]);
                    if (16 * rb + mine < n_q) {
                        float* const p = out + (16 * rb + mine) * n_keys + t0 + c;
                        if constexpr (THROUGH) stream_store_at(p, v);
                        else *reinterpret_cast<floatx4u*>(p) = v;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            } else if (query < n_q) {
                if (t0 + KEYS <= n_keys) {                  // uniform
#pragma unroll
                    for (int b = 0; b < BK; ++b) {
                        if constexpr (THROUGH) stream_store_at(row + 16 * b, w[rb][b]);
                        else *reinterpret_cast<floatx4u*>(row + 16 * b) = w[rb][b];
                    }
                } else {
#pragma unroll
                    for (int b = 0; b < BK; ++b)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (16 * b + i < mine) row[16 * b + i] = w[rb][b][i];
                }
            }
        }
    }
}

// n_q <= 8 / 16 / 32
template <int D, bool WIDE, bool THROUGH>
auto kernel_of(int n_q) {
    return n_q <= 8    ? srft_scores_kernel<D, 1, WIDE, false, THROUGH>
           : n_q <= 16 ? srft_scores_kernel<D, 1, WIDE, true, THROUGH>
                       : srft_scores_kernel<D, 2, WIDE, true, THROUGH>;
}

template <int D>
int launch(const srft_plan* p, const void* q, int n_q, const uint8_t* codes, const float* scales, long long n_keys, float* out,
           hipStream_t st) {
    // a workgroup per tile, up to one per compute unit, two at d = 64 with up to 16 queries (what the registers hold at once; at
    // d = 128 a second workgroup that waits for the first only adds its own start: 1,000,000 keys, 8 queries 21.5 us against
    // 25.5; d = 64, 32 queries, 300,000 keys 11 against 14)
    const int keys = n_q <= 16 ? kTileKeys<D, 1> : kTileKeys<D, 2>;
    const long long n_tiles = (n_keys + keys - 1) / keys;
    long long grid = p->max_wgs > 0 ? p->max_wgs : (D == 64 && n_q <= 16 ? 2 : 1) * p->compute_units;
    if (grid > n_tiles) grid = n_tiles;
    const bool wide = p->gw > 1;
    // Rows of whole 64-byte pieces, halves of a line, are written through (device_util.h).  Over three / six sets of keys and scores in turn,
    // left to the L2 -> written through: 8 queries at d = 128, 100,000 keys 4.85 -> 4.5 us, 400,000 10.3 -> 9.6 / 10.8 -> 9.7, 1,000,000 22.5 ->
    // 22.5 / 23.9 -> 23.9; 16 queries, 1,000,000 29.3 -> 24.8 / 29.5 -> 31.3; 32 queries, 100,000 8.0 -> 6.3, 1,000,000 43.9 -> 38.1 / 43.7 -> 44.4; d =
    // 64, 8 queries, 400,000 8.0 -> 6.6, 1,000,000 14.0 -> 13.4 / 17.9 -> 18.9.  Pieces that straddle lines are not (334,146 keys 16.5 -> 24.7), nor a
    // single row, which is next to nothing to write back (1,000,000 keys at d = 128 17.0 -> 17.3).
    const bool through = n_q > 1 && n_keys % 16 == 0 && (reinterpret_cast<uintptr_t>(out) & 63) == 0;
    const auto kernel = through ? (wide ? kernel_of<D, true, true>(n_q) : kernel_of<D, false, true>(n_q))
                                : (wide ? kernel_of<D, true, false>(n_q) : kernel_of<D, false, false>(n_q));
    return srft_launch(kernel, dim3((unsigned)grid), 64 * kWaves, st, (const uint4*)q, n_q, (const uint4*)p->q_table,
                       (int)(p->transform == SRFT_TRANSFORM_HADAMARD), codes, scales, p->gw, n_keys, out);
}

}  // namespace

int srft_launch_scores(const srft_plan* p, const void* q, int n_q, const uint8_t* codes, const float* scales,
                       long long n_keys, float* out, hipStream_t st) {
    switch (p->d) {
        case 64: return launch<64>(p, q, n_q, codes, scales, n_keys, out, st);
        case 128: return launch<128>(p, q, n_q, codes, scales, n_keys, out, st);
        case 192: return launch<192>(p, q, n_q, codes, scales, n_keys, out, st);
        case 256: return launch<256>(p, q, n_q, codes, scales, n_keys, out, st);
        default: return SRFT_ERR_BAD_D;
    }
}
