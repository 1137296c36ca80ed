// rotated_queries.h -- device code shared by the kernels that contract queries against the stored codes
// (kernels/scores.hip, kernels/decode_attention.hip).
#ifndef SRFT_ROTATED_QUERIES_H
#define SRFT_ROTATED_QUERIES_H
#include "device_util.h"

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

// ---- the transform of the queries: a Cooley-Tukey FFT in fp32 (or the Walsh-Hadamard butterflies), D = 16 L points, 16
// points per lane
struct srft_cf { float x, y; };
__device__ __forceinline__ srft_cf operator+(srft_cf a, srft_cf b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ srft_cf operator-(srft_cf a, srft_cf b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ srft_cf srft_mul(srft_cf a, srft_cf b) { return {fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x)}; }
constexpr float srft_cos48(int k) {                          // cos(2 pi k / 48)
    constexpr double c[13] = {1.0, 0.99144486137381041, 0.96592582628906829, 0.92387953251128674, 0.86602540378443865, 0.79335334029123517,
                              0.70710678118654752, 0.60876142900872064, 0.5, 0.38268343236508977, 0.25881904510252076,
                              0.13052619222005159, 0.0};
    k %= 48;
    if (k > 24) k = 48 - k;
    return (float)(k > 12 ? -c[24 - k] : c[k]);
}
template <int E>                                             // times exp(-2 pi i E / 48)
__device__ __forceinline__ srft_cf srft_turn(srft_cf a) {
    if constexpr (E % 48 == 0) return a;
    else if constexpr (E % 48 == 12) return {a.y, -a.x};
    else if constexpr (E % 48 == 24) return {-a.x, -a.y};
    else if constexpr (E % 48 == 36) return {-a.y, a.x};
    else return srft_mul(a, {srft_cos48(E), -srft_cos48(E + 36)});           // (sin t = cos(t - quarter turn))
}
__device__ __forceinline__ void srft_dft4(srft_cf a, srft_cf b, srft_cf c, srft_cf d, srft_cf& x0, srft_cf& x1, srft_cf& x2, srft_cf& x3) {
    const srft_cf s0 = a + c, s1 = a - c, s2 = b + d, s3 = b - d;
    x0 = s0 + s2;
    x2 = s0 - s2;
    x1 = {s1.x + s3.y, s1.y - s3.x};
    x3 = {s1.x - s3.y, s1.y + s3.x};
}
// in[j] -> out[k] = sum_j in[j] exp(-2 pi i j k / L), L = 4 B: j = B a + b, k = m + 4 q
template <int L>
__device__ __forceinline__ void srft_dft(const srft_cf (&in)[L], srft_cf (&out)[L]) {
    constexpr int B = L / 4;
    srft_cf t[B][4];
#pragma unroll
    for (int b = 0; b < B; ++b) srft_dft4(in[b], in[B + b], in[2 * B + b], in[3 * B + b], t[b][0], t[b][1], t[b][2], t[b][3]);
    constexpr int S = 48 / L;
    if constexpr (B > 1) {
        t[1][1] = srft_turn<S>(t[1][1]);
        t[1][2] = srft_turn<2 * S>(t[1][2]);
        t[1][3] = srft_turn<3 * S>(t[1][3]);
    }
    if constexpr (B > 2) {
        t[2][1] = srft_turn<2 * S>(t[2][1]);
        t[2][2] = srft_turn<4 * S>(t[2][2]);
        t[2][3] = srft_turn<6 * S>(t[2][3]);
    }
    if constexpr (B > 3) {
        t[3][1] = srft_turn<3 * S>(t[3][1]);
        t[3][2] = srft_turn<6 * S>(t[3][2]);
        t[3][3] = srft_turn<9 * S>(t[3][3]);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        if constexpr (B == 1) {
            out[m] = t[0][m];
        } else if constexpr (B == 2) {
            out[m] = t[0][m] + t[1][m];
            out[m + 4] = t[0][m] - t[1][m];
        } else if constexpr (B == 3) {
            const srft_cf s = t[1][m] + t[2][m], d = t[1][m] - t[2][m];
            constexpr float r = srft_cos48(4);               // sqrt(3) / 2
            const srft_cf h = {fmaf(s.x, -0.5f, t[0][m].x), fmaf(s.y, -0.5f, t[0][m].y)};
            out[m] = t[0][m] + s;
            out[m + 4] = {fmaf(d.y, r, h.x), fmaf(d.x, -r, h.y)};
            out[m + 8] = {fmaf(d.y, -r, h.x), fmaf(d.x, r, h.y)};
        } else {
            srft_dft4(t[0][m], t[1][m], t[2][m], t[3][m], out[m], out[m + 4], out[m + 8], out[m + 12]);
        }
    }
}
// 16 real values -> the coefficients 0 .. 8 of their DFT
__device__ __forceinline__ void srft_real_dft16(const float (&x)[16], srft_cf (&out)[9]) {
    float r[4], u[4];
    srft_cf t[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const float e = x[b] + x[8 + b], o = x[4 + b] + x[12 + b];
        r[b] = e + o;
        u[b] = e - o;
        t[b] = {x[b] - x[8 + b], x[12 + b] - x[4 + b]};
    }
    t[1] = srft_turn<3>(t[1]);
    t[2] = srft_turn<6>(t[2]);
    t[3] = srft_turn<9>(t[3]);
    out[0] = {(r[0] + r[2]) + (r[1] + r[3]), 0.0f};
    out[8] = {(r[0] + r[2]) - (r[1] + r[3]), 0.0f};
    out[4] = {r[0] - r[2], r[3] - r[1]};
    srft_cf c9, c13;
    srft_dft4(t[0], t[1], t[2], t[3], out[1], out[5], c9, c13);
    out[7] = {c9.x, -c9.y};
    out[3] = {c13.x, -c13.y};
    constexpr float q = srft_cos48(6);                       // sqrt(1/2)
    const float d = q * (u[1] - u[3]), s = q * (u[1] + u[3]);
    out[2] = {u[0] + d, -u[2] - s};
    out[6] = {u[0] - d, u[2] - s};
}
template <int L>
__device__ __forceinline__ void srft_wht(float (&x)[L]) {
#pragma unroll
    for (int h = 1; h < L; h *= 2)
#pragma unroll
        for (int i = 0; i < L; ++i)
            if (!(i & h)) {
                const float a = x[i], b = x[i + h];
                x[i] = a + b;
                x[i + h] = a - b;
            }
}

// The operands of 16 RB queries for a workgroup of W wavefronts: q'_p = z_p / max(lambda_p, 1e-6), z the packed transform
// (Eq. 1-2) of the query, split into fp16 hi + lo.  qs: [block of 16][group][hi, lo][64 lanes]: lane l holds query l % 16
// and the 8 codes of unit l / 16 of the group, in the order decode8 lays them out (element e <-> code e / 2 + 4 (e % 2)).
// Queries past n_q are zero.
//
// Every workgroup does this for itself (a launch of its own took 3.0 us at d = 128, 4.6 us at d = 256), so what counts is its
// latency, and as a product with the dense matrix that was the 64 KB (d = 128) or 256 KB (d = 256) that a compute unit had
// to pull in: 5,400 of the 12,200 clocks of the decode attention's scan over 1000 keys at d = 128, 12,500 of 26,300 at
// d = 256.  As an FFT it reads the query and 80 bytes per lane.  n = L i + j: lane (query, j) transforms its 16 values over i
// (real, 9 coefficients k1), turns them by exp(-2 pi i j k1 / D); lane (query, k1) transforms over j, which gives the bins
// k1 + 16 k2 (past D / 2: the conjugates of D - k); then every thread scales and splits a unit of 8.  The three exchanges go
// through LDS.
// us, against the matrix: scores of 8 queries, 300,000 keys at d = 256 15.2 -> 13.0, 1,000,000 at d = 64 14.2 -> 13.5, 32
// queries, 300,000 keys at d = 128 13.2 -> 12.5; decode attention of 4 queries, 4096 keys at d = 256 15.5 -> 14.3, d = 192
// 13.3 -> 12.2.  Error against 64 bits 1.7e-7 -> 1.2e-7 (scores at d = 256), 1.3e-7 -> 1.1e-7 (d = 128).
// table: [L] x 5 units of 16 bytes: exp(-2 pi i j k1 / D) for k1 = 1 .. 8, then the signs of n = L i + j (bit i); then D floats:
// the packing constant (1 / sqrt(D) or sqrt(2 / D)) / max(lambda_p, 1e-6).
// Everything is multiplied by factor (1 or -1).  `fetch` is called when the loads of the queries and the table are on their
// way, for the caller's own: their wait does not include it.
// scratch: srft_query_scratch_bytes bytes of LDS, 16-byte aligned, free again on return (all wavefronts have passed a barrier).
template <int D, int RB> constexpr int kQueryMid = 16 * RB * 9 * (D / 16 + 1) * 8;       // bytes: [query][k1][j], padded
template <int D> constexpr int kQueryRow = D + 12;           // floats: [query][p], padded (9 bins of 5 queries side by side, 4 channels of 16
                                                             // queries on different banks); [D] takes what nobody reads
template <int D, int RB>
constexpr int srft_query_scratch_bytes() {
    return kQueryMid<D, RB> + 16 * RB * kQueryRow<D> * 4;
}
template <int D, int W, int RB, class F>
__device__ __forceinline__ void
srft_query_operands(const uint4* __restrict__ q, int n_q, int q0, const uint4* __restrict__ table, int hadamard, float factor,
                    unsigned char* scratch, uint4* qs, F fetch) {
    constexpr int L = D / 16, G = D / 32, U = D / 8, NT = 64 * W, PER = (16 * RB * U + NT - 1) / NT;     // PER: units per thread
    static_assert(L % 4 == 0 && L <= 16 && 16 * RB * L <= NT && kQueryMid<D, RB> % 16 == 0, "a thread per (query, j)");
    const int tid = threadIdx.x, nq = min(16 * RB, n_q - q0), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool first_step = 64 * wave < nq * L, last_step = 64 * wave < 16 * RB * U;     // wavefronts that have a part in them
    float* const mid = reinterpret_cast<float*>(scratch);
    float* const z = reinterpret_cast<float*>(scratch + kQueryMid<D, RB>);
    // (threads without a query repeat the last one's loads; wavefronts of them have none: 8 wavefronts of 23 loads held the
    // tiles' loads back by 2000 clocks)
    const int j = tid % L, mine = min(tid / L, nq - 1);
    const unsigned short* const xq = reinterpret_cast<const unsigned short*>(q) + (size_t)(q0 + mine) * D + j;
    uint32_t raw[16], signs = 0;
    floatx4 tw[4], mul[PER][2];
    if (first_step) {
#pragma unroll
        for (int i = 0; i < 16; ++i) raw[i] = xq[L * i];
#pragma unroll
        for (int i = 0; i < 4; ++i) tw[i] = reinterpret_cast<const floatx4*>(table)[5 * j + i];
        signs = reinterpret_cast<const uint32_t*>(table)[20 * j + 16];
    }
    if (last_step)
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int e = 0; e < 2; ++e) mul[i][e] = reinterpret_cast<const floatx4*>(table)[5 * L + 2 * ((tid + NT * i) / 16 % U) + e];
    __builtin_amdgcn_sched_barrier(0);
    fetch();
    __builtin_amdgcn_sched_barrier(0);
    float x[16];
    if (first_step) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            x[i] = (float)__builtin_bit_cast(_Float16, (unsigned short)(raw[i] ^ (((signs >> i) & 1u) << 15)));
    }
    if (hadamard) {                                          // uniform; k = L i' + j'
        if constexpr ((D & (D - 1)) == 0) {
            if (tid < nq * L) {
                srft_wht(x);
#pragma unroll
                for (int i = 0; i < 16; ++i) mid[(mine * 16 + i) * (L + 1) + j] = x[i];
            }
            __syncthreads();
            if (tid < nq * 16) {
                float y[L];
#pragma unroll
                for (int i = 0; i < L; ++i) y[i] = mid[tid * (L + 1) + i];
                srft_wht(y);
#pragma unroll
                for (int i = 0; i < L; ++i) z[tid / 16 * kQueryRow<D> + L * (tid % 16) + i] = y[i];
            }
        }
    } else {
        srft_cf* const m = reinterpret_cast<srft_cf*>(mid);
        if (tid < nq * L) {
            srft_cf a[9];
            srft_real_dft16(x, a);
#pragma unroll
            for (int k = 1; k < 9; ++k) a[k] = srft_mul(a[k], {tw[(k - 1) / 2][2 * ((k - 1) % 2)], tw[(k - 1) / 2][2 * ((k - 1) % 2) + 1]});
#pragma unroll
            for (int k = 0; k < 9; ++k) m[(mine * 9 + k) * (L + 1) + j] = a[k];
        }
        __syncthreads();
        if (tid < nq * 9) {
            srft_cf in[L], out[L];
#pragma unroll
            for (int i = 0; i < L; ++i) in[i] = m[tid * (L + 1) + i];
            srft_dft<L>(in, out);
            const int k1 = tid % 9;
            float* const up = z + tid / 9 * kQueryRow<D> + k1;
            float* const down = z + tid / 9 * kQueryRow<D> - k1;
            // (in this order: the imaginary part of bin 0 lands where the real part of bin D / 2 goes, behind it, and that
            // of bin D / 2 at [D]; bins that a lane has twice, k1 = 0 and 8, are written twice)
#pragma unroll
            for (int k = 0; k < L / 2; ++k) {
                up[16 * k] = out[k].x;
                up[16 * k + D / 2] = out[k].y;
            }
#pragma unroll
            for (int k = L / 2; k < L; ++k) {
                down[16 * (L - k)] = out[k].x;
                down[16 * (L - k) + D / 2] = -out[k].y;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        // (16 neighbouring lanes have the 16 queries of a block: the other way round their writes all hit the same banks)
        const int at = tid + NT * i, u = at / 16 % U, query = at % 16 + at / (16 * U) * 16;
        if (16 * RB * U % NT == 0 || query < 16 * RB) {
            const float* const row = z + query * kQueryRow<D> + 8 * u;
            const floatx4 lo4 = *reinterpret_cast<const floatx4*>(row), hi4 = *reinterpret_cast<const floatx4*>(row + 4);
            half8 hi, lo;
#pragma unroll
            for (int e = 0; e < 8; ++e) {                    // element e <-> code e / 2 + 4 (e % 2)
                const float v = query < nq ? (e % 2 ? hi4 : lo4)[e / 2] * mul[i][e % 2][e / 2] * factor : 0.0f;
                hi[e] = (_Float16)v;
                lo[e] = (_Float16)(v - (float)hi[e]);
            }
            uint4* const dst = qs + ((query / 16 * G + u / 4) * 2) * 64 + 16 * (u % 4) + query % 16;
            dst[0] = __builtin_bit_cast(uint4, hi);
            dst[64] = __builtin_bit_cast(uint4, lo);
        }
    }
    __syncthreads();
}

#endif  // SRFT_ROTATED_QUERIES_H
