// One decode step of attention over the stored records: out_i = sum_t softmax_t(softmax_scale <q_i, k_t>) v_t.
//
// Both products are taken in the rotated domain on the codes (kernels/scores.hip, kernels/attend.hip): a score is
// <q'_i, code_t * scale_t> with q' = Q (s * q) / max(lambda_k, 1e-6), the output is one inverse transform per query of
// sum_t w_t code_t * scale_t.  Two launches:
//
// 1. srft_attention_scan_kernel: ONE pass over K and V.  A workgroup forms q' (every workgroup for itself); a wavefront takes
//    tiles of 64 or 32 keys: scores, a softmax running over its own tiles (its maximum, the sum of its weights; sums taken
//    under an older maximum are scaled down when the maximum grows), weighted sums of the V codes.  The wavefronts of a
//    workgroup meet in LDS at the end, and a workgroup leaves n_q x D sums, a maximum and a sum of weights per query.
// 2. srft_attention_finish_kernel: the workgroups' sums are brought under one maximum, added in a fixed order (the result does
//    not depend on timing), divided by the sum of the weights and taken through the inverse transform.
//
// What bounds it: at 131,072 keys and d = 128 the record is 21 MB (4 us at the rate of a copy) and every wavefront of the chip
// has one tile, so the time is the latency of the launches and of one tile's chain (about 18,400 clocks in the scan: 5,800 until
// q' has reached every wavefront, 1,000 more until the tile is in LDS, 2,800 scores, 800 softmax, 2,200 values, 5,100 to meet,
// 3,000 of them with the wait for the slowest wavefront).  Scores and weights therefore never leave the registers: with keys on
// the rows and queries on the columns of the score product, a lane holds, for ITS query (lane % 16), the keys of its quarter of
// the wavefront (lane / 16), which is what the second product takes as its B operand and what a running maximum and its
// correction need; with channels on the rows and queries on the columns of the second product the sums belong to the same query.
// Measured, us, against a scan that stores the scores, a value pass over 2048 one-wavefront workgroups and two reductions:
// d = 128, 8 queries, 131,072 keys 36.6 -> 13.6, 400,000 keys 51 -> 23; 32 queries, 400,000 keys 111 -> 38; d = 256, 4 queries,
// 4096 keys 27.7 -> 9.15; d = 64, 1 query, 500 keys 21.9 -> 10.5.  Error against 64 bits 6e-6 -> 4e-7.
#include <algorithm>

#include "../rotated_queries.h"

namespace {

constexpr int kWaves = 8;                                    // wavefronts per workgroup of the scan: two per SIMD
constexpr int kScanGridMax = 1024;                           // most workgroups of the scan (a cap on the grid may ask for more than one per unit)
constexpr float kLowest = -3.0e38f;                          // "no key yet": finite, so that differences of two are

typedef int v2i __attribute__((ext_vector_type(2)));


// maximum / sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (one query's quarters), in all of them
__device__ __forceinline__ float quarters_max(float m) {
    const uint2 a = swap16(__float_as_uint(m), __float_as_uint(m));
    m = fmaxf(__uint_as_float(a.x), __uint_as_float(a.y));
    return other_half_max(m);
}
__device__ __forceinline__ float quarters_sum(float s) {
    const uint2 a = swap16(__float_as_uint(s), __float_as_uint(s));
    s = __uint_as_float(a.x) + __uint_as_float(a.y);
    const uint2 b = swap32(__float_as_uint(s), __float_as_uint(s));
    return __uint_as_float(b.x) + __uint_as_float(b.y);
}

// over the 64 lanes, in all of them; the order of the sum is fixed
template <int CTRL> __device__ __forceinline__ float row_rotated(float x) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, row_rotated<0x128>(x));                     // row_ror: 8, 4, 2, 1 within 16 lanes
    x = fmaxf(x, row_rotated<0x124>(x));
    x = fmaxf(x, row_rotated<0x122>(x));
    x = fmaxf(x, row_rotated<0x121>(x));
    return quarters_max(x);
}
__device__ __forceinline__ float wave_sum(float x) {
    x += row_rotated<0x128>(x);
    x += row_rotated<0x124>(x);
    x += row_rotated<0x122>(x);
    x += row_rotated<0x121>(x);
    return quarters_sum(x);
}

// D: head dimension.  KEYS: keys per tile, 64 or 32 (then ONE, but at D = 192).  WIDE: groups of gw > 1 runs of 32 channels share a scale.
// blockIdx.y: block of 16 queries.  (Both blocks of 32 queries in one wavefront -- the codes decoded once -- needs more
// registers than two wavefronts per SIMD leave: 250 spilled at d = 128.)
// ONE: no wavefront has more than one tile (up to 131,072 keys and 16 queries on a whole chip): nothing is asked for behind
// it and nothing scaled down (and 110 registers do where 201 did, d = 128).  us: 8 queries, 131,072 keys at d = 128 13.8 ->
// 13.6, at d = 256 22.9 -> 22.4; 16 queries, 9000 keys at d = 256 15.3 -> 15.0; 8 queries, 60,000 keys at d = 192 15.0 ->
// 14.75.
// TEAM: wavefronts to a tile, each with D / 32 / TEAM groups of it on both sides.  With few tiles most of a workgroup's wavefronts
// had none, and the chain of one tile, a third of it vector instructions of one wavefront, was what the scan took (4096 keys at
// d = 256: 2,100 clocks scores, 2,300 values, 1,200 the sums' way to the workspace, of 11,400).  The members add up their shares
// of the scores in LDS, in one order, so all hold the same scores and weights, and their sums of the values are of different
// channels: nothing is left to meet for.  us, a wavefront to a tile -> teams: 4 queries, 4096 keys at d = 256 10.45 -> 9.15, 500 9.25
// -> 7.95, 12,000 13.9 -> 12.65; of two wavefronts, 20,000 14.05 -> 13.65, 16 queries, 30,000 15.95 -> 14.45; d = 192, 8 queries,
// 5000 10.95 -> 10.05, 16,000 12.05 -> 11.15; d = 128, 2000 7.5 -> 7.05, 9000 9.65 -> 8.85, 30,000 9.35 -> 9.05.
template <int D, int KEYS, bool WIDE, bool ONE, int TEAM = 1>
__global__ void __launch_bounds__(64 * kWaves, 2)
srft_attention_scan_kernel(const uint4* __restrict__ q, int n_q, const uint4* __restrict__ q_table,
                           int hadamard, float q_sign, const uint8_t* __restrict__ k_codes,
                           const float* __restrict__ k_scales, int k_gw, const uint8_t* __restrict__ v_codes,
                           const float* __restrict__ v_scales, int v_gw, long long n_keys, float softmax_scale,
                           float* __restrict__ part, float* __restrict__ part_max, float* __restrict__ part_sum) {
    constexpr int ALL = D / 32, G = ALL / TEAM;              // groups of a row, and of those this wavefront's
    constexpr int QUADS = G / 4, REST = G % 4;               // its part of a row of codes: QUADS x 64 bytes, then REST x 16 bytes
    constexpr int W = kWaves, TEAMS = W / TEAM;
    constexpr int ROW = D / 2, MINE = 16 * G;                // bytes of a row, of the part
    constexpr int BK = KEYS / 16;                            // blocks of 16 keys
    constexpr int KQ = KEYS / 4;                             // keys per quarter of the wavefront
    constexpr int VROW = MINE + 16;                          // padded: the 16 rows of a transposed read hit different banks
    constexpr int VTILE = KEYS * VROW + 4 * 8;               // and 8 bytes more per quarter's rows keep the quarters apart
    constexpr int NV = KEYS * G / 64;                        // 16-byte pieces of a V tile per lane
    constexpr int NB = 2 * G;                                // blocks of 16 channels
    constexpr int WAVE_BYTES = VTILE + (2 * G + 1) * KEYS * 4;
    constexpr int TILE_BYTES = W * WAVE_BYTES, MEET_BYTES = TEAMS * 16 * (D + 4) * 4, QUERY_BYTES = srft_query_scratch_bytes<D, 1>();
    constexpr int LDS_BYTES = TEAM == 1 ? TILE_BYTES : std::max(TILE_BYTES, std::max(MEET_BYTES, QUERY_BYTES));
    static_assert(D % 64 == 0 && VTILE % 16 == 0 && (KEYS == 32 || KEYS == 64), "layout");
    static_assert(TEAM == 1 || (ONE && KEYS == 32 && (G == 2 || G == 4) && G * TEAM == ALL), "a team has one tile, two or four groups a wavefront");
    static_assert(KEYS == 64 || ONE || D == 192, "tiles of 32 keys are for short prefixes");
    __shared__ __align__(16) unsigned char lds[LDS_BYTES];
    __shared__ uint4 qs[ALL * 2 * 64];
    __shared__ float meet[2][W][16];
    __shared__ floatx4 shares[TEAM > 1 ? W : 1][TEAM > 1 ? KEYS / 16 : 1][TEAM > 1 ? 64 : 1];    // of the scores, per wavefront

    // all arguments in one go: loaded where they are used, each is a round trip of its own in the chain of one tile
    asm volatile("" :: "s"(hadamard), "s"(q_sign), "s"(softmax_scale), "s"(part), "s"(part_max), "s"(part_sum), "s"(q_table),
                 "s"(k_codes), "s"(k_scales), "s"(v_codes), "s"(v_scales), "s"(n_keys));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);    // (uniform: tile addresses in scalar registers)
    const int l16 = lane & 15, a = lane >> 4;                // query (or key / channel of a block of 16), quarter
    const int team = wave / TEAM, member = wave % TEAM, g0 = member * G;     // (wavefronts left over: a team that has no tile)
    unsigned char* const vt = lds + wave * WAVE_BYTES;       // this wavefront's V tile and scales: no other one touches them
    float* const ks = reinterpret_cast<float*>(vt + VTILE);  // [group][key]
    float* const vs = ks + G * KEYS;
    float* const vtop = vs + G * KEYS;                       // [key]: largest of V's scales
    const int q0 = 16 * blockIdx.y, nq = min(16, n_q - q0);  // the queries of this workgroup

    const long long n_tiles = (n_keys + KEYS - 1) / KEYS;
    const long long stride = (long long)gridDim.x * TEAMS;
    // tiles team * grid + workgroup + k * stride: a short prefix is spread over as many compute units as it has tiles
    const long long first = (long long)team * gridDim.x + blockIdx.x;

    // Which key a lane loads as row m = l16 of block b of the K tile: KQ (m / 4) + 4 b + m % 4.  The score product's result
    // register i of quarter a is row 4 a + i, so a quarter ends up with the keys KQ a .. KQ a + KQ - 1 (register [b][i]:
    // key KQ a + 4 b + i), and the transposed reads of V take whole rows of keys per quarter.
    uint4 pk[BK][QUADS ? QUADS : 1], pv[NV];
    static_assert(REST == 0 || REST == 2, "d is a multiple of 64");
    uint2 pr[BK];
    floatx4 pks[(G + 3) / 4], pvs[(G + 3) / 4];
    auto fetch_scales = [&](floatx4 (&dst)[(G + 3) / 4], const float* src, int gw, long long t0, int rl) __attribute__((always_inline)) {
        if constexpr (WIDE) {
            const int ns = ALL / gw;
#pragma unroll
            for (int j = 0; j < G; ++j) dst[j / 4][j % 4] = (src + t0 * ns)[(unsigned)(rl * ns + (g0 + j) / gw)];
        } else {
            const float* row = src + t0 * ALL + (unsigned)(rl * ALL + g0);
#pragma unroll
            for (int j = 0; j + 4 <= G; j += 4) dst[j / 4] = *reinterpret_cast<const floatx4u*>(row + j);
#pragma unroll
            for (int j = G / 4 * 4; j < G; ++j) dst[j / 4][j % 4] = row[j];
        }
    };
    // keys past the end alias to the last one
    auto lim_of = [&](long long t0) __attribute__((always_inline)) { return (int)min((long long)(KEYS - 1), n_keys - 1 - t0); };
    auto fetch_k = [&](long long tile, bool all) __attribute__((always_inline)) {
        const long long t0 = tile * KEYS;
        const int lim = all ? lim_of(t0) : 0;
        const uint8_t* kb = k_codes + t0 * ROW + 16 * g0;
#pragma unroll
        for (int b = 0; b < BK; ++b) {
            const unsigned row = (unsigned)min(KQ * (l16 >> 2) + 4 * b + (l16 & 3), lim) * ROW;
#pragma unroll
            for (int s = 0; s < QUADS; ++s) pk[b][s] = *reinterpret_cast<const uint4*>(kb + (row + 64 * s + 16 * a));
            if constexpr (REST > 0) pr[b] = *reinterpret_cast<const uint2*>(kb + (row + 64 * QUADS + 8 * a));
        }
        fetch_scales(pks, k_scales, k_gw, t0, min(lane & (KEYS - 1), lim));
    };
    auto fetch_v = [&](long long tile, bool all) __attribute__((always_inline)) {
        const long long t0 = tile * KEYS;
        const int lim = all ? lim_of(t0) : 0;
        const uint8_t* vb = v_codes + t0 * ROW + 16 * g0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int u = lane + 64 * i;
            pv[i] = *reinterpret_cast<const uint4*>(vb + ((unsigned)min(u / G, lim) * ROW + 16 * (u % G)));
        }
        fetch_scales(pvs, v_scales, v_gw, t0, min(lane & (KEYS - 1), lim));
    };
    auto v_at = [&](int row) __attribute__((always_inline)) { return vt + row * VROW + (row / KQ) * 8; };

    // ---- the operands of the queries, while the first tile is on its way
    static_assert(srft_query_scratch_bytes<D, 1>() <= LDS_BYTES, "the tiles' LDS serves it first");
    srft_query_operands<D, W, 1>(q, n_q, q0, q_table, hadamard, q_sign, lds, qs, [&]() __attribute__((always_inline)) {
        fetch_k(min(first, n_tiles - 1), first < n_tiles);
        fetch_v(min(first, n_tiles - 1), first < n_tiles);
    });

    floatx4 acc[NB];                                         // [block of 16 channels]: channels 16 b + 4 a + i, query l16
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = floatx4{0, 0, 0, 0};
    float top = kLowest, den = 0.0f;                         // maximum of the exponents, sum of weights
    // The products weight * scale go to the matrix cores as fp16 hi + lo, and neither may leave fp16's range: a query's weights
    // are taken times 2^fit, which brings the largest product that its sums hold (big, under the present maximum; a key's
    // largest scale stands for all of them) to 2^13 .. 2^14.  What a product below it loses is then under 2^-37 of the largest,
    // whatever the scales and weights of other keys, before or after.  The sums carry the same power, divided out at the end.
    // (A power from the largest scale alone, that only fell, cost up to 1 % less at 400,000 keys and more, and left a key beside
    // or after one of 2^28 times its scale and no weight with 1e-3 of error.)
    float big = 0.0f;
    int fit = 113;
    // weights are 2^(c * score - top)
    const float c = softmax_scale * 1.44269504088896340736f;

    // The LDS operands of a step are read one step ahead of their use.
    struct KStep { uint4 h, l; float4 sc[BK]; };
    auto load_k = [&](KStep& f, int j) __attribute__((always_inline)) {
        f.h = qs[((g0 + j) * 2 + 0) * 64 + lane];
        f.l = qs[((g0 + j) * 2 + 1) * 64 + lane];
#pragma unroll
        for (int b = 0; b < BK; ++b) f.sc[b] = *reinterpret_cast<const float4*>(&ks[j * KEYS + KQ * a + 4 * b]);
    };
    struct VStep { v2i r[2]; float4 sc[BK]; };
    auto load_v = [&](VStep& f, int j) __attribute__((always_inline)) {
        // transposed reads of the group's two 16-channel units: lane l gives the address of key row KQ a + l16 (mod KQ) and
        // receives, as nibbles, the 16 rows' codes of channel l16
#pragma unroll
        for (int h = 0; h < 2; ++h)
            f.r[h] = __builtin_amdgcn_ds_read_tr4_b64_v2i32(
                (__attribute__((address_space(3))) v2i*)(v_at(KQ * a + (l16 & (KQ - 1))) + 8 * (2 * j + h)));
#pragma unroll
        for (int b = 0; b < BK; ++b) f.sc[b] = *reinterpret_cast<const float4*>(&vs[j * KEYS + KQ * a + 4 * b]);
    };
    float w[BK][4];                                          // scores, then weights: keys KQ a + 4 b + i of query l16
    const auto scores = [&](const long long tile, const bool more) __attribute__((always_inline)) {
        // LDS of one wavefront: its accesses complete in program order
#pragma unroll
        for (int j = 0; j < G; ++j) {
            ks[j * KEYS + (lane & (KEYS - 1))] = pks[j / 4][j % 4];
            vs[j * KEYS + (lane & (KEYS - 1))] = pvs[j / 4][j % 4];
        }
        float most = fabsf(pvs[0][0]);
#pragma unroll
        for (int j = 1; j < G; ++j) most = fmaxf(most, fabsf(pvs[j / 4][j % 4]));
        vtop[lane & (KEYS - 1)] = most;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int u = lane + 64 * i;
            unsigned char* dst = v_at(u / G) + 16 * (u % G);
            reinterpret_cast<uint2*>(dst)[0] = make_uint2(pv[i].x, pv[i].y);         // (8-byte aligned)
            reinterpret_cast<uint2*>(dst)[1] = make_uint2(pv[i].z, pv[i].w);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // The next tile goes into the registers that have just been read.  Not under a branch (the compiler then keeps both
        // sets: 100 registers more at d = 128): past the end every lane reads the first row of this tile again.
        if constexpr (!ONE) fetch_v(more ? tile + stride : tile, more);
        // ---- scores: keys on the rows, queries on the columns
#pragma unroll
        for (int b = 0; b < BK; ++b) {
#pragma unroll
            for (int s = 0; s < QUADS; ++s) pk[b][s] = srft_quad_transpose(pk[b][s]);
            if constexpr (REST > 0) pr[b] = srft_pair_transpose(pr[b]);
        }
        KStep kc, kn;
        load_k(kc, 0);
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (j + 1 < G) load_k(kn, j + 1);
            const half8 qh = __builtin_bit_cast(half8, kc.h), ql = __builtin_bit_cast(half8, kc.l);
#pragma unroll
            for (int b = 0; b < BK; ++b) {
                const uint4& four = pk[b][j / 4 < QUADS ? j / 4 : 0];
                const uint32_t kd = j >= 4 * QUADS ? (j == 4 * QUADS ? pr[b].x : pr[b].y)
                                  : j % 4 == 0 ? four.x : j % 4 == 1 ? four.y : j % 4 == 2 ? four.z : four.w;
                const half8 kf = __builtin_bit_cast(half8, decode8(kd));
                const float scv[4] = {kc.sc[b].x, kc.sc[b].y, kc.sc[b].z, kc.sc[b].w};
                floatx4 s = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qh, floatx4{0, 0, 0, 0}, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, ql, s, 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 4; ++i) w[b][i] = j == 0 ? s[i] * scv[i] : fmaf(s[i], scv[i], w[b][i]);
            }
            kc = kn;
            // one group's operands at a time (registers), or two where they allow it
            if ((KEYS == 64 && !ONE) || j % 2) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!ONE) fetch_k(more ? tile + stride : tile, more);
    };
    const auto values = [&](const long long tile) __attribute__((always_inline)) {
        VStep vc, vn;
        load_v(vc, 0);
        // ---- running softmax, per query (column)
        {
            float m = w[0][0];
#pragma unroll
            for (int v = 1; v < KQ; ++v) m = fmaxf(m, w[v / 4][v % 4]);
            m = fmaxf(quarters_max(m) * c, kLowest);
            const float t = fmaxf(m, top), down = __builtin_amdgcn_exp2f(top - t);
            top = t;
            den *= down;
#pragma unroll
            for (int v = 0; v < KQ; ++v) w[v / 4][v % 4] = __builtin_amdgcn_exp2f(fmaf(c, w[v / 4][v % 4], -top));
            if (tile == n_tiles - 1) {                       // uniform: keys past the end weigh nothing
                int lim = lim_of(tile * KEYS);
                asm volatile("" : "+s"(lim));                 // (the comparisons stay here, out of the way of the first tile)
#pragma unroll
                for (int v = 0; v < KQ; ++v) w[v / 4][v % 4] = KQ * a + v <= lim ? w[v / 4][v % 4] : 0.0f;
            }
#pragma unroll
            for (int v = 0; v < KQ; ++v) den += w[v / 4][v % 4];
            float product = 0.0f;
#pragma unroll
            for (int b = 0; b < BK; ++b) {
                const float4 f = *reinterpret_cast<const float4*>(&vtop[KQ * a + 4 * b]);
                product = fmaxf(product, fmaxf(fmaxf(w[b][0] * f.x, w[b][1] * f.y), fmaxf(w[b][2] * f.z, w[b][3] * f.w)));
            }
            big = fmaxf(big * down, quarters_max(product));
            const int fit_now = 140 - max((int)((__float_as_uint(big) >> 23) & 0xFF), 27);    // 13 - exponent, at most 113
            const float change = __builtin_ldexpf(down, fit_now - fit);
            fit = fit_now;
            if (!ONE && tile != first && __ballot(change != 1.0f))           // uniform
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] *= change;
#pragma unroll
            for (int v = 0; v < KQ; ++v) w[v / 4][v % 4] = __builtin_ldexpf(w[v / 4][v % 4], fit);
        }
        // ---- sums of the values: channels on the rows, queries on the columns; k-step s takes the keys 8 s .. 8 s + 7 of
        // every quarter, in the order 0 4 1 5 2 6 3 7 of decode8
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (j + 1 < G) load_v(vn, j + 1);
            half8 wh[BK / 2], wl[BK / 2];
#pragma unroll
            for (int s = 0; s < BK / 2; ++s) {
                // w * scale as fp16 hi (truncated) + fp16 lo of the exact remainder: about 21 bits
                const float4 f0 = vc.sc[2 * s], f1 = vc.sc[2 * s + 1];
                const float sc0[4] = {f0.x, f0.y, f0.z, f0.w}, sc1[4] = {f1.x, f1.y, f1.z, f1.w};
                uint32_t hh[4], ll[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float x0 = w[2 * s][i] * sc0[i], x1 = w[2 * s + 1][i] * sc1[i];
                    const auto h2 = __builtin_amdgcn_cvt_pkrtz(x0, x1);
                    const auto l2 = __builtin_amdgcn_cvt_pkrtz(fmaf((float)h2[0], -1.0f, x0), fmaf((float)h2[1], -1.0f, x1));
                    hh[i] = __builtin_bit_cast(uint32_t, h2);
                    ll[i] = __builtin_bit_cast(uint32_t, l2);
                }
                wh[s] = __builtin_bit_cast(half8, make_uint4(hh[0], hh[1], hh[2], hh[3]));
                wl[s] = __builtin_bit_cast(half8, make_uint4(ll[0], ll[1], ll[2], ll[3]));
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                floatx4& sum = acc[2 * j + h];
#pragma unroll
                for (int s = 0; s < BK / 2; ++s) {
                    const half8 f = __builtin_bit_cast(half8, decode8((uint32_t)(s == 0 ? vc.r[h].x : vc.r[h].y)));
                    sum = __builtin_amdgcn_mfma_f32_16x16x32_f16(f, wh[s], sum, 0, 0, 0);
                    sum = __builtin_amdgcn_mfma_f32_16x16x32_f16(f, wl[s], sum, 0, 0, 0);
                }
            }
            vc = vn;
            if ((KEYS == 64 && !ONE) || j % 2) __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    if constexpr (TEAM > 1) {
        if (first < n_tiles) {
            scores(first, false);
#pragma unroll
            for (int b = 0; b < BK; ++b) shares[wave][b][lane] = floatx4{w[b][0], w[b][1], w[b][2], w[b][3]};
        }
        __syncthreads();
        if (first < n_tiles) {
            floatx4 s[BK];                                   // the members' shares in their order: all of them get the same scores
#pragma unroll
            for (int b = 0; b < BK; ++b) s[b] = shares[team * TEAM][b][lane];
#pragma unroll
            for (int k = 1; k < TEAM; ++k)
#pragma unroll
                for (int b = 0; b < BK; ++b) s[b] += shares[team * TEAM + k][b][lane];
#pragma unroll
            for (int b = 0; b < BK; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) w[b][i] = s[b][i];
            values(first);
        }
    } else {
        for (long long tile = first; tile < n_tiles; tile += stride) {
            scores(tile, tile + stride < n_tiles);
            values(tile);
            if constexpr (ONE) break;
        }
    }
    // ---- the teams of the workgroup that had a tile meet
    const int active = (int)min((long long)TEAMS, (n_tiles - 1 - blockIdx.x) / gridDim.x + 1);
    den = quarters_sum(den);
    if (member == 0 && team < TEAMS && a == 0) {
        meet[0][team][l16] = top;
        meet[1][team][l16] = den;
    }
    float* const dst = part + ((size_t)blockIdx.x * n_q + q0) * D;
    if (active == 1) {                                       // nobody to meet (short prefixes: 2200 clocks at d = 256 otherwise)
        if (team == 0) {
            const float f = __builtin_ldexpf(1.0f, -fit);
            if (tid < nq) {
                part_max[(q0 + l16) * kScanGridMax + blockIdx.x] = top;
                part_sum[(q0 + l16) * kScanGridMax + blockIdx.x] = den;
            }
            if (l16 < nq)
#pragma unroll
                for (int b = 0; b < NB; ++b) *reinterpret_cast<floatx4*>(&dst[l16 * D + 32 * g0 + 16 * b + 4 * a]) = acc[b] * f;
        }
        return;
    }
    __syncthreads();
    float t = meet[0][0][l16];                               // (teams without a tile: kLowest and 0)
#pragma unroll
    for (int k = 1; k < TEAMS; ++k) t = fmaxf(t, meet[0][k][l16]);
    const float f = __builtin_ldexpf(__builtin_amdgcn_exp2f(top - t), -fit);
    if (tid < nq) {
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k < TEAMS; ++k) s = fmaf(meet[1][k][l16], __builtin_amdgcn_exp2f(meet[0][k][l16] - t), s);
        part_max[(q0 + l16) * kScanGridMax + blockIdx.x] = t;
        part_sum[(q0 + l16) * kScanGridMax + blockIdx.x] = s;
    }
    if constexpr (TEAM > 1) {                                // sums: [team][query][channel]
        float* const merge = reinterpret_cast<float*>(lds);
        constexpr int MROW = D + 4;                          // padded
        __syncthreads();                                     // (the tiles have been read)
        if (team < active && l16 < nq)
#pragma unroll
            for (int b = 0; b < NB; ++b) *reinterpret_cast<floatx4*>(&merge[(team * nq + l16) * MROW + 32 * g0 + 16 * b + 4 * a]) = acc[b] * f;
        __syncthreads();
        for (int e = tid; e < nq * (D / 4); e += 64 * W) {
            const int r = e / (D / 4), p = e % (D / 4);
            floatx4 s = *reinterpret_cast<const floatx4*>(&merge[r * MROW + 4 * p]);
            for (int k = 1; k < active; ++k) s += *reinterpret_cast<const floatx4*>(&merge[(k * nq + r) * MROW + 4 * p]);
            *reinterpret_cast<floatx4*>(&dst[r * D + 4 * p]) = s;
        }
        return;
    }
    // (a wavefront to a tile) sums: [wavefront][query][channel], as many channels at a time as fit
    float* const merge = reinterpret_cast<float*>(lds);
    static_assert(W * 16 * (16 + 4) * 4 <= LDS_BYTES, "at least one block at a time");
    int nb = NB;
    while (active * nq * (16 * nb + 4) * 4 > LDS_BYTES) nb = (nb + 1) / 2;
    const int mrow = 16 * nb + 4;                            // padded
    for (int b0 = 0; b0 < NB; b0 += nb) {
        const int b1 = min(NB, b0 + nb);
        if (b0) __syncthreads();
        if (wave < active && l16 < nq)
#pragma unroll
            for (int b = 0; b < NB; ++b)
                if (b >= b0 && b < b1)                       // uniform
                    *reinterpret_cast<floatx4*>(&merge[(wave * nq + l16) * mrow + 16 * (b - b0) + 4 * a]) = acc[b] * f;
        __syncthreads();
        const auto add = [&](int r, int p) __attribute__((always_inline)) {      // 16-byte piece p of query r
            const float* const from = &merge[r * mrow + 4 * p];
            floatx4 s = *reinterpret_cast<const floatx4*>(from);
            if (active == W) {                               // (all reads on their way together)
#pragma unroll
                for (int k = 1; k < W; ++k) s += *reinterpret_cast<const floatx4*>(from + k * nq * mrow);
            } else {
                for (int k = 1; k < active; ++k) s += *reinterpret_cast<const floatx4*>(from + k * nq * mrow);
            }
            *reinterpret_cast<floatx4*>(&dst[r * D + 16 * b0 + 4 * p]) = s;
        };
        const int per = 4 * (b1 - b0);
        if (per == 4 * NB)                                   // (a division by a constant)
            for (int e = tid; e < nq * 4 * NB; e += 64 * W) add(e / (4 * NB), e % (4 * NB));
        else
            for (int e = tid; e < nq * per; e += 64 * W) add(e / per, e % per);
    }
}

// Workgroup (query, block of 64 outputs), 1024 threads.  It adds the scan's workgroups over all D channels (thread: channels
// 4 (t % (D / 4)) .. + 3 of the workgroups t / (D / 4), + SLICES, ...), then takes its 64 columns of the inverse transform
// (thread: outputs 4 (t % 16) .. + 3, terms KS (t / 16) ...).  Every load is on its way before the first is waited for, the
// maxima ahead of the sums ahead of the matrix.  Bound by what one compute unit can pull in: 64 columns instead of all D
// leave a quarter of the matrix at d = 256 (64 of 256 KB) for the same sums (128 KB).  Against a workgroup per query that
// reduced the maxima through LDS: 5.6 -> 4.0 us at d = 128, 256 workgroups to add; 6.7 -> 5.8 us at d = 256, 128 of them.
// A workgroup's maximum reaches the threads that add its sums from the lane that holds it (a load for each was 256 loads of one
// value per workgroup); with the scan's shorter end, d = 128, 131,072 keys 15.3 -> 14.1 us, d = 256, 4096 keys 14.3 -> 12.7.
// AHEAD: rows of sums a thread asks for at once, for 64, 128 or 256 (D = 192: 63, 126, 252) workgroups to add in one pass;
// what is not needed costs as much as what is (4096 keys at d = 256, 128 of them, 12.8 -> 12.0 us; a branch around each load
// 0.3 us where all are needed).
template <int D, int AHEAD>
__global__ void __launch_bounds__(1024)
srft_attention_finish_kernel(const float* __restrict__ part, const float* __restrict__ part_max,
                             const float* __restrict__ part_sum, int parts, int n_q, const float4* __restrict__ rmat,
                             float* __restrict__ out) {
    constexpr int C4 = D / 4, SLICES = 1024 / C4, KS = D / 64;
    constexpr bool HELD = D != 192;                          // the lanes hold the maxima of the workgroups whose sums are on their way
    constexpr int PM = HELD ? SLICES * AHEAD / 64 : 4;       // of 64 PM workgroups
    static_assert(!HELD || PM * 64 == SLICES * AHEAD, "whole wavefronts of them");
    constexpr int ROWS = D == 192 ? SLICES : 16;             // partial sums that meet in LDS (else one per wavefront)
    __shared__ __align__(16) float red[ROWS * D];
    __shared__ __align__(16) float accs[D];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, query = blockIdx.x;
    const int c4 = tid % C4, slice = tid / C4;
    // every wavefront finds the maximum and the sum of the weights for itself
    float pm[PM], ps[PM];
    auto load_max = [&](int p0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PM; ++i) {
            const int p = min(p0 + 64 * i + lane, parts - 1);
            pm[i] = part_max[query * kScanGridMax + p];
            ps[i] = p0 + 64 * i + lane < parts ? part_sum[query * kScanGridMax + p] : 0.0f;
        }
    };
    floatx4 x[AHEAD];
    float xm[HELD ? 1 : AHEAD];
    auto load = [&](int base) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int p = min(base + slice + i * SLICES, parts - 1);
            if constexpr (!HELD) xm[i] = part_max[query * kScanGridMax + p];
            x[i] = *reinterpret_cast<const floatx4*>(part + ((size_t)p * n_q + query) * D + 4 * c4);
        }
    };
    load_max(0);
    load(0);
    float4 m[KS];
#pragma unroll
    for (int i = 0; i < KS; ++i) m[i] = rmat[(KS * (tid / 16) + i) * C4 + 16 * blockIdx.y + tid % 16];
    float top = kLowest;
    for (int p0 = 0; p0 < parts; p0 += 64 * PM) {            // (one pass but where a cap asks for more than 256 workgroups)
        if (p0) load_max(p0);
#pragma unroll
        for (int i = 0; i < PM; ++i) top = fmaxf(top, pm[i]);
    }
    top = wave_max(top);
    float den = 0.0f;
    for (int p0 = 0; p0 < parts; p0 += 64 * PM) {
        if (parts > 64 * PM) load_max(p0);
#pragma unroll
        for (int i = 0; i < PM; ++i) den = fmaf(ps[i], __builtin_amdgcn_exp2f(pm[i] - top), den);
    }
    den = wave_sum(den);
    floatx4 sum = {0, 0, 0, 0};
    for (int base = 0; base < parts; base += AHEAD * SLICES) {               // (uniform: lanes read each other's maxima)
        const int p0 = base + slice;
        if (base > 0) load(base);
        if (HELD && parts > 64 * PM) load_max(base);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            float its;
            if constexpr (HELD)                              // workgroup p0 + i SLICES: lane p % 64 of register p / 64 % PM
                its = __shfl(pm[i * SLICES / 64], (slice + i * SLICES) & 63);
            else
                its = xm[i];
            const float f = p0 + i * SLICES < parts ? __builtin_amdgcn_exp2f(its - top) : 0.0f;
            sum = f != 0.0f ? sum + x[i] * f : sum;          // (a workgroup that counts for nothing may hold anything)
        }
    }
    if constexpr (D == 128) {                                // two slices in a wavefront
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint2 h = swap32(__float_as_uint(sum[e]), __float_as_uint(sum[e]));
            sum[e] = __uint_as_float(h.x) + __uint_as_float(h.y);
        }
    } else if constexpr (D == 64) {                          // four
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] = quarters_sum(sum[e]);
    }
    if (D != 192 || slice < SLICES)
        *reinterpret_cast<floatx4*>(&red[(D == 192 ? slice : wave) * D + 4 * c4]) = sum;     // (lanes with the same sum: the same value)
    __syncthreads();
    if (tid < D) {
        float v = red[tid];
#pragma unroll
        for (int k = 1; k < ROWS; ++k) v += red[k * D + tid];
        accs[tid] = v;
    }
    __syncthreads();
    floatx4 o = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < KS; ++i) {
        const float v = accs[KS * (tid / 16) + i];
        o[0] = fmaf(m[i].x, v, o[0]);
        o[1] = fmaf(m[i].y, v, o[1]);
        o[2] = fmaf(m[i].z, v, o[2]);
        o[3] = fmaf(m[i].w, v, o[3]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = quarters_sum(o[e]);   // the wavefront's four sets of terms
    if (lane < 16) *reinterpret_cast<floatx4*>(&red[wave * 64 + 4 * lane]) = o;      // (red has been read: the barrier above)
    __syncthreads();
    if (tid < 64) {
        float v = red[tid];
#pragma unroll
        for (int k = 1; k < 16; ++k) v += red[k * 64 + tid];
        out[(size_t)query * D + 64 * blockIdx.y + tid] = v / den;
    }
}

template <int D>
int launch(const srft_plan* pk, const srft_plan* pv, const void* q, int n_q, const uint8_t* k_codes, const float* k_scales,
           const uint8_t* v_codes, const float* v_scales, long long n_keys, float softmax_scale, float* out, void* workspace,
           hipStream_t st) {
    // Tiles of 64 keys, or of 32 where that still leaves every wavefront of the chip at most one (and then wavefronts in teams, while
    // every team has at most one): the chain of one tile is then half as long.  Workgroups: one per tile, up to one per compute unit
    // (its eight wavefronts fill the register file); with two blocks of queries half of that each, so that both read a tile at about
    // the same time.
    const int blocks = n_q <= 16 ? 1 : 2;
    long long most = pv->compute_units;
    if (pk->max_wgs > 0) most = pk->max_wgs;
    if (pv->max_wgs > 0 && (pk->max_wgs == 0 || pv->max_wgs < most)) most = pv->max_wgs;
    long long grid = std::max(most / blocks, 1LL);           // (a cap is on all of them; one for each block of queries is the least)
    if (grid > kScanGridMax) grid = kScanGridMax;
    // (63, 126 or 252 are what the finish adds in one pass at D = 192: 8192 keys, 8 queries 14.2 -> 12.4 us)
    const auto in_one_pass = [](long long n) {
        if (D == 192)
            for (const long long one_pass : {63, 126, 252})
                if (n > one_pass && n <= one_pass + one_pass / 63) return one_pass;
        return n;
    };
    // What 252 of 256 leave over of the short tiles, 64,513 to 65,536 keys at D = 192, goes to a few wavefronts as a second one (65,000
    // keys, 1 / 8 / 16 queries 14.6 / 15.8 / 17.5 us; 64-key tiles 16.6 / 16.9 / 17.5, 256 workgroups and a finish of two passes 15.7 / 17.0 /
    // 18.9); with two blocks of queries 64-key tiles are the faster (32,768 keys, 17 queries 15.9, so 16.2).
    const long long cut = in_one_pass(grid);
    const bool narrow = n_keys <= 32 * kWaves * (blocks == 1 ? grid : cut);
    grid = cut;
    const long long n_tiles = narrow ? (n_keys + 31) / 32 : (n_keys + 63) / 64;
    grid = in_one_pass(std::min(grid, n_tiles));
    static_assert((size_t)kScanGridMax * 32 * (2 + D) <= srft_attend_workspace_floats(D), "fits what callers are told to bring");
    float* part_max = (float*)workspace;                     // [32][kScanGridMax] each
    float* part_sum = part_max + kScanGridMax * 32;
    float* part = part_sum + kScanGridMax * 32;              // [workgroup][n_q][D]
    const float sign = softmax_scale < 0.0f ? -1.0f : 1.0f;  // goes into the queries: the kernel's scale is not negative
    const auto pick = [&](auto shared, auto plain) { return pk->gw > 1 || pv->gw > 1 ? shared : plain; };
    // as many wavefronts to a tile (two groups each, or four) as leaves every team at most one
    constexpr int TWO = D / 64, FOUR = D == 256 ? 2 : 1;
    const auto kernel =
        narrow && n_tiles <= kWaves / TWO * grid    ? pick(srft_attention_scan_kernel<D, 32, true, true, TWO>, srft_attention_scan_kernel<D, 32, false, true, TWO>)
        : narrow && n_tiles <= kWaves / FOUR * grid ? pick(srft_attention_scan_kernel<D, 32, true, true, FOUR>, srft_attention_scan_kernel<D, 32, false, true, FOUR>)
        : narrow && n_tiles <= kWaves * grid        ? pick(srft_attention_scan_kernel<D, 32, true, true>, srft_attention_scan_kernel<D, 32, false, true>)
        : narrow                                    ? pick(srft_attention_scan_kernel<D, 32, true, D != 192>, srft_attention_scan_kernel<D, 32, false, D != 192>)
        : n_tiles <= kWaves * grid                  ? pick(srft_attention_scan_kernel<D, 64, true, true>, srft_attention_scan_kernel<D, 64, false, true>)
                                                    : pick(srft_attention_scan_kernel<D, 64, true, false>, srft_attention_scan_kernel<D, 64, false, false>);
    const int rc = srft_launch(kernel, dim3((unsigned)grid, blocks), 64 * kWaves, st, (const uint4*)q, n_q, (const uint4*)pk->q_table,
                               (int)(pk->transform == SRFT_TRANSFORM_HADAMARD), sign, k_codes, k_scales, pk->gw, v_codes, v_scales,
                               pv->gw, n_keys, sign * softmax_scale, part, part_max, part_sum);
    if (rc != SRFT_OK) return rc;
    constexpr int A = D / 16, most_at_once = D == 192 ? 252 : 256;
    const auto finish = grid <= most_at_once / 4   ? srft_attention_finish_kernel<D, A / 4>
                        : grid <= most_at_once / 2 ? srft_attention_finish_kernel<D, A / 2>
                                                   : srft_attention_finish_kernel<D, A>;
    return srft_launch(finish, dim3((unsigned)n_q, D / 64), 1024, st, (const float*)part, (const float*)part_max, (const float*)part_sum,
                       (int)grid, n_q, (const float4*)pv->rmat_f32, out);
}

}  // namespace

int srft_launch_decode_attention(const srft_plan* pk, const srft_plan* pv, const void* q, int n_q, const uint8_t* k_codes,
                                 const float* k_scales, const uint8_t* v_codes, const float* v_scales, long long n_keys,
                                 float softmax_scale, float* out, void* workspace, hipStream_t st) {
    switch (pv->d) {
        case 64: return launch<64>(pk, pv, q, n_q, k_codes, k_scales, v_codes, v_scales, n_keys, softmax_scale, out, workspace, st);
        case 128: return launch<128>(pk, pv, q, n_q, k_codes, k_scales, v_codes, v_scales, n_keys, softmax_scale, out, workspace, st);
        case 192: return launch<192>(pk, pv, q, n_q, k_codes, k_scales, v_codes, v_scales, n_keys, softmax_scale, out, workspace, st);
        case 256: return launch<256>(pk, pv, q, n_q, k_codes, k_scales, v_codes, v_scales, n_keys, softmax_scale, out, workspace, st);
        default: return SRFT_ERR_BAD_D;
    }
}
