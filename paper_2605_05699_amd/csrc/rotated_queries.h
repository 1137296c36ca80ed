// rotated_queries.h -- device code shared by the kernels that contract queries against the stored codes
// (kernels/scores.hip, kernels/decode_attention.hip).
#ifndef SRFT_ROTATED_QUERIES_H
#define SRFT_ROTATED_QUERIES_H
#include "device_util.h"

typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));     // scales and scores are 4-byte aligned

__device__ __forceinline__ uint2 swap16(uint32_t a, uint32_t b) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    return make_uint2(r[0], r[1]);
}
__device__ __forceinline__ uint2 swap32(uint32_t a, uint32_t b) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    return make_uint2(r[0], r[1]);
}
// 16 bytes that quarter k of the wavefront (lane / 16) loaded whole from group k of a quad of groups -> dword k of each of the
// four groups, in quarter k: a 4 x 4 transpose over the quarters.
__device__ __forceinline__ uint4 srft_quad_transpose(const uint4& r) {
    const uint2 x01 = swap16(r.x, r.y), x23 = swap16(r.z, r.w);
    const uint2 y02 = swap32(x01.x, x23.x), y13 = swap32(x01.y, x23.y);
    return make_uint4(y02.x, y13.x, y02.y, y13.y);
}

// 8 bytes that quarter k loaded from two groups (its dwords 2 k and 2 k + 1 of their eight) -> dword k of each, in quarter k.
__device__ __forceinline__ uint2 srft_pair_transpose(const uint2& r) {
    const uint2 x = swap16(r.x, r.y);
    return swap32(x.x, x.y);
}

// The operands of 16 RB queries for a workgroup of W wavefronts: q' = w / (lambda max(lambda, 1e-6)) with w the write path's
// transform (its dense matrix, fp16 hi + lo, one slab of 32 channels per wavefront or PARTS wavefronts), split into
// fp16 hi + lo.  qs: [block of 16][group][hi, lo][64 lanes]: lane l holds query l % 16 and the 8 codes of unit l / 16 of the
// group, in the order decode8 lays them out (element e <-> code e / 2 + 4 (e % 2)).  Queries past n_q are zero.
// Every workgroup does this for itself (64 KB of matrix from L2 at d = 128, 256 KB at d = 256); a launch of its own took
// 3.0 us at d = 128, 4.6 us at d = 256.  `fetch` is called when the operands' loads are on their way, for the caller's own:
// their wait does not include it.  scratch: srft_query_scratch_bytes bytes of LDS, free again on return (all wavefronts
// have passed a barrier).
template <int D, int W, int RB>
constexpr int srft_query_scratch_bytes() {
    return 16 * RB * (D * 2 + 16) + (D / 32) * ((W / (D / 32) > 0 ? W / (D / 32) : 1) - 1) * 32 * RB * 16 * 4;
}
template <int D, int W, int RB, class F>
__device__ __forceinline__ void
srft_query_operands(const uint4* __restrict__ q, int n_q, int q0, const uint4* __restrict__ wfrag,
                    const float* __restrict__ q_scale, float unscale, unsigned char* scratch, uint4* qs, F fetch) {
    constexpr int G = D / 32, PARTS = W / G > 0 ? W / G : 1, T = D / 16 / PARTS;     // T: MFMA k-steps per wavefront
    static_assert(PARTS * T * 16 == D && (RB == 1 || RB == 2) && G <= W, "every slab has its wavefronts");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = RB == 2 ? lane & 31 : lane & 15;       // query (RB == 1: columns 16 .. 31 repeat 0 .. 15)
    const bool holds = RB == 2 || (lane & 16) == 0;
    const int slab = min(wave / PARTS, G - 1), piece = wave % PARTS;
    const bool spare = wave / PARTS >= G;                    // (D = 192: the last wavefronts repeat a slab and keep it to themselves)
    floatx16 qacc = floatx16{0};
    floatx4 q_mul[4];                                        // 1 / (lambda max(lambda, 1e-6)) of this lane's 16 channels
    {
        // the queries meet the matrix through LDS: every wavefront needs all of them
        constexpr int XROW = D * 2 + 16;
        for (int i = tid; i < 16 * RB * (D / 8); i += 64 * W)
            *reinterpret_cast<uint4*>(scratch + (i / (D / 8)) * XROW + 16 * (i % (D / 8))) =
                q[(size_t)min(q0 + i / (D / 8), n_q - 1) * (D / 8) + i % (D / 8)];
        const unsigned char* xr = scratch + col * XROW + 16 * (2 * piece * T + half);
        const uint4* wr = wfrag + ((size_t)(slab * (D / 16) + piece * T) * 2) * 64 + lane;
        constexpr int TB = T < 4 ? T : T % 8 == 0 ? 8 : 4;   // k-steps in flight
#pragma unroll
        for (int t0 = 0; t0 < T; t0 += TB) {
            uint4 h[TB], l[TB];
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                h[t] = wr[(2 * (t0 + t)) * 64];
                l[t] = wr[(2 * (t0 + t) + 1) * 64];
            }
            if (t0 + TB >= T) {
#pragma unroll
                for (int i = 0; i < 4; ++i) q_mul[i] = reinterpret_cast<const floatx4*>(q_scale)[8 * slab + 4 * half + i];
                __builtin_amdgcn_sched_barrier(0);
                fetch();
                __builtin_amdgcn_sched_barrier(0);
            }
            if (t0 == 0) __syncthreads();
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                const half8 b = *reinterpret_cast<const half8*>(xr + 32 * (t0 + t));
                qacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, h[t]), b, qacc, 0, 0, 0);
                qacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, l[t]), b, qacc, 0, 0, 0);
            }
        }
    }
    // (used under a branch only: without this the loads move there, behind the caller's)
    asm volatile("" : "+v"(q_mul[0]), "+v"(q_mul[1]), "+v"(q_mul[2]), "+v"(q_mul[3]));
    if constexpr (PARTS > 1) {
        constexpr int SLOTS = 32 * RB;
        float* sums = reinterpret_cast<float*>(scratch + 16 * RB * (D * 2 + 16)) + (slab * (PARTS - 1) + piece - 1) * (SLOTS * 16) +
                      16 * RB * half + col;
        if (piece > 0 && holds)
#pragma unroll
            for (int v = 0; v < 16; ++v) sums[v * SLOTS] = qacc[v];
        __syncthreads();
        if (piece == 0)
#pragma unroll
            for (int k = 1; k < PARTS; ++k)
#pragma unroll
                for (int v = 0; v < 16; ++v) qacc[v] += sums[k * (SLOTS * 16) + v * SLOTS];
    }
    if (!spare && piece == 0 && holds) {
        // lane (query col, half) holds the 16 channels 32 slab + 16 half + v: two whole units
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            half8 hi, lo;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int v = 8 * i + (e / 2) + 4 * (e % 2);
                const float x = q0 + col < n_q ? (qacc[v] * unscale) * q_mul[v / 4][v % 4] : 0.0f;
                hi[e] = (_Float16)x;
                lo[e] = (_Float16)(x - (float)hi[e]);
            }
            uint4* dst = qs + (((col >> 4) * G + slab) * 2) * 64 + 16 * (2 * half + i) + (col & 15);
            dst[0] = __builtin_bit_cast(uint4, hi);
            dst[64] = __builtin_bit_cast(uint4, lo);
        }
    }
    __syncthreads();
}

#endif  // SRFT_ROTATED_QUERIES_H
