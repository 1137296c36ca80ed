// device_util.h -- device-side helpers shared by the kernel templates.
#ifndef SRFT_DEVICE_UTIL_H
#define SRFT_DEVICE_UTIL_H

#include <type_traits>

#include "common.h"
#include "launch_shape.h"

// Stores of results, which go through to memory (sc1) instead of staying in the L2 of a die.  What bounds a launch of up to some
// 100 MB is not the rate of its loop alone but the write-back of the L2s at its end: each die's is searched and written back before
// the next launch, and beyond some 16 MB of results lines are also evicted one by one while the kernel reads.  Written through,
// nothing is left to write back.  Only for stores that cover whole lines, or halves of 64 bytes: a part of one goes to memory as a partial
// write (8-bit records at d = 256, 16 bytes of a row at a time: 62 -> 130 us over 300 MB).  By sizes and alignment each path has a rule
// where it pays (srft_write_staged, srft_fold_through, srft_read_through in launch_shape.h; scores.hip).  us by bytes moved, non-temporal stores -> sc1
// nt:
//   read, d = 128   11 MB 5.4 -> 4.3   22 6.1 -> 5.4   33 9.7 -> 7.8   44 13.4 -> 11.6   88 21.5 -> 21.8   352 65.8 -> 64.7
//   read, d = 256   11 MB 6.2 -> 5.3   33 11.3 -> 9.8  44 15.4 -> 12.6 88 24.2 -> 24.0   176 41.8 -> 40.6
//   read, d = 96    10 MB 6.0 -> 4.5   31 10.1 -> 8.2  83 22.0 -> 21.5 330 65.5 -> 63.9
//   write, d = 256  11 MB 5.8 -> 5.3   33 10.7 -> 9.7  88 22.0 -> 19.0 176 37.8 -> 36.3   352 70.2 -> 68.5
//   write, d = 128  11 MB 5.3 -> 5.0   30 9.15 -> 8.8  (beyond 60 MB left to the L2)
// nt on top of sc1 keeps the lines out of the memory-side cache: better from 100 MB on (reads 67.0 -> 65.0 at 352 MB) and for d = 64 and
// 96 wherever memory is cold (130 MB at d = 64 33.3 -> 28.9), worse where the sets in turn just fill that cache (three of 88 MB at d = 128
// 20.5 -> 21.8).  Stored without it: all scales (a tile has
// 512 bytes of them at d = 128; with it 14 plans x 50 vectors 3.3 -> 3.5).
// The buffer form of the store takes the policy as an operand; base is uniform, offsets in bytes stay below 2^31.
constexpr int kStoreThrough = 16, kStoreThroughOnce = 18;                // cache policy: sc1; sc1 nt
__device__ __forceinline__ auto stream_rows(void* base) { return __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00027000); }
template <int POLICY = kStoreThroughOnce, class T>
__device__ __forceinline__ void stream_store(T* base, unsigned at, uint4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), stream_rows(base), (int)(at * sizeof(T)), 0, POLICY);
}
template <int POLICY = kStoreThroughOnce, class T>
__device__ __forceinline__ void stream_store(T* base, unsigned at, uint2 v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), stream_rows(base), (int)(at * sizeof(T)), 0, POLICY);
}
// (lanes with there = false store behind the buffer's end, which the hardware drops: no branch)
template <int POLICY = kStoreThroughOnce>
__device__ __forceinline__ void stream_store(float* base, unsigned at, float v, bool there = true) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), stream_rows(base), there ? (int)(at * 4) : (int)0x80000000, 0, POLICY);
}
// A row's piece written through, or left to the L2 (nt alone).
template <bool THROUGH, class T>
__device__ __forceinline__ void store_row(T* base, unsigned at, uint4 v) {
    if constexpr (THROUGH) stream_store(base, at, v);
    else __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), reinterpret_cast<u32x4*>(base + at));
}
// ... at any address of four-byte alignment.  The data registers of a store of more than 8 bytes must not be written again by a
// vector instruction within two wait states.  The compiler keeps to that behind its own stores and does not see into this one, so the
// wait states stand with it.  (Nor does it count the store: its waits for loads then include it.)
__device__ __forceinline__ void stream_store_at(float* p, floatx4 v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
// Non-temporal loads help where one load instruction covers whole cache lines (the read path's code units) and cost up to 20 %
// where several loads of a lane share a line (the folded write paths, whose lanes read 32 or 64 contiguous bytes), so those loads
// stay plain.
__device__ __forceinline__ uint4 stream_load(const uint4* p) {
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)));
}
__device__ __forceinline__ uint2 stream_load(const uint2* p) {
    return __builtin_bit_cast(uint2, __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p)));
}

// ------------------------------------------------------------------------------------------
// device helpers
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float other_half_max(float m) {
    // lanes l and l^32 hold the two halves of one vector's group: one v_permlane32_swap.
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Make the loop-invariant matrix fragments "used" here, so that the wait for their loads is placed
// before the main loop and not inside it (where it would also wait for the loop's own prefetches).
template <int N>
__device__ __forceinline__ void hold_in_registers(half8 (&a)[N], half8 (&b)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(a[i]), "+v"(b[i]));
}
template <int N, int M>
__device__ __forceinline__ void hold_in_registers(half8 (&a)[N][M], half8 (&b)[N][M]) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < M; ++j) asm volatile("" : "+v"(a[i][j]), "+v"(b[i][j]));
}

// The instruction arbiter of a compute unit favours its oldest wavefronts: of the workgroups that share a unit the
// one dispatched first ran 25 % ahead of the others and left the unit early, while the kernel waited for the
// last one.  Every workgroup therefore walks through the four wavefront priorities, one per stage, offset by its
// place in the dispatch order: over four stages each has held each priority once, and they finish together
// (end times of the workgroups 440..620 us -> 565..600 us at d = 128, 8 M vectors; launches 1.5-3.5 % shorter).  Not used
// where two workgroups per unit take turns on one accumulator set (the folded write path at d = 256), which measured 1 %
// slower with it.
__device__ __forceinline__ void rotate_priority(int stage) {
    switch (((int)(blockIdx.x * 4 / gridDim.x) + stage) & 3) {
        case 0: __builtin_amdgcn_s_setprio(0); break;
        case 1: __builtin_amdgcn_s_setprio(1); break;
        case 2: __builtin_amdgcn_s_setprio(2); break;
        default: __builtin_amdgcn_s_setprio(3); break;
    }
}

template <int N> struct Accs;          // one 32x32 accumulator tile per slab, as named registers
template <> struct Accs<1> { floatx16 a; };
template <> struct Accs<2> { floatx16 a, b; };
template <class F> __device__ __forceinline__ void each_acc(Accs<1>& p, F f) { f(p.a, 0); }
template <class F> __device__ __forceinline__ void each_acc(Accs<2>& p, F f) { f(p.a, 0); f(p.b, 1); }

// Eight values already multiplied by 1/scale -> eight two's-complement nibbles in one dword.
// Adding 1.5*2^23 + 8 rounds to nearest-even and leaves q + 8 (1..15) in the low four bits above a
// constant bit pattern; a shift-add chain concatenates the nibbles (no borrows because q + 8 > 0),
// the constant is subtracted once and flipping bit 3 of each nibble turns q + 8 into q mod 16.
__device__ __forceinline__ uint32_t shl4_add(uint32_t p, uint32_t x) {
    uint32_t r;                                  // (p << 4) + x as ONE instruction (the compiler prefers shift + 3-way add)
    asm("v_lshl_add_u32 %0, %1, 4, %2" : "=v"(r) : "v"(p), "v"(x));
    return r;
}
__device__ __forceinline__ uint32_t pack8(const floatx16& acc, int base, float inv) {
    constexpr float kMagic = 12582912.0f + 8.0f;
    constexpr uint32_t kMagicBits = 0x4B400000u;
    uint32_t p = __float_as_uint(fmaf(acc[base + 7], inv, kMagic));
#pragma unroll
    for (int i = 6; i >= 0; --i) p = shl4_add(p, __float_as_uint(fmaf(acc[base + i], inv, kMagic)));
    uint32_t k = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) k += kMagicBits << (4 * i);
    return (p - k) ^ 0x88888888u;
}

// Four values already multiplied by 1/scale -> four two's-complement bytes in one dword (8-bit output).
// Adding 1.5 * 2^23 rounds to nearest-even and leaves q mod 256 in the low byte of the bit pattern.
__device__ __forceinline__ uint32_t pack4_bytes(const floatx16& acc, int base, float inv) {
    constexpr float kMagic = 12582912.0f;
    const uint32_t a = __float_as_uint(fmaf(acc[base], inv, kMagic)), b = __float_as_uint(fmaf(acc[base + 1], inv, kMagic));
    const uint32_t c = __float_as_uint(fmaf(acc[base + 2], inv, kMagic)), d = __float_as_uint(fmaf(acc[base + 3], inv, kMagic));
    const uint32_t lo = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);       // byte 0 of a, byte 0 of b, 0, 0
    const uint32_t hi = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
    return (hi << 16) | lo;
}

// What a workgroup of a batched launch works on: its segment, and its place among that segment's workgroups.  Lane l compares
// boundary l of the (ascending) table, so one load and one ballot find it whatever the number of segments (a scan of the
// table took 50 ns per segment in front of everything else: a read launch of 64 plans x 32 vectors 7.7 -> 5.7 us).
// Workgroups are dealt to the 8 accelerator dies round robin, each die with an L2 of its own; here a die takes a
// contiguous eighth of the list, so that the workgroups of one plan share one copy of its matrix table instead of pulling
// it into every L2.  Measured against workgroup b = place b: 64 plans x 512 vectors at d = 96, write 6.8 -> 5.8 us;
// 52 x 4096 at d = 256, read 40.6 -> 36.6 us; 56 x 8192 at d = 128, write 37.3 -> 36.6 us; 4 x 1,048,576 within 0.5 %.  Over
// 2 to 64 plans and 5 to 600 MB at d = 96, 128, 256: reads 0 to 33 % and writes 0 to 33 % shorter, most where a plan has few
// tiles; at 2 and 3 plans with one to two tiles a workgroup it lost up to 10 % until such segments were cut where the dies
// meet (launch_shape.h).
struct srft_work {
    const uint4* frag;
    const void* in;
    void* out;
    float* scales;
    long long n_vec;
    float unscale;
    int blocks, place;              // workgroups of the segment, this one's place among them
};
__device__ __forceinline__ int srft_block_by_die() {
    const int q = gridDim.x >> 3, r = gridDim.x & 7, die = blockIdx.x & 7;
    return die * q + min(die, r) + (int)(blockIdx.x >> 3);                   // a permutation of 0 .. gridDim.x - 1
}
template <bool WRITE, int N>
__device__ __forceinline__ srft_work srft_work_of_block(const srft_batch<N>& a) {
    static_assert(N <= 64 && (N & (N - 1)) == 0, "a lane per boundary");
    const int block = srft_block_by_die();
    if constexpr (N == 0) {                                  // segments of one length, a constant step apart
        const int i = srft_even_segment(block, a.shape), start = srft_even_start(i, a.shape);
        const srft_plan_entry* e = reinterpret_cast<const srft_plan_entry*>(reinterpret_cast<const char*>(a.plan) + i * a.plan_step);
        return {(const uint4*)(const __attribute__((address_space(1))) uint4*)e->table[WRITE ? 0 : 1], a.in + i * a.in_step, a.out + i * a.out_step,
                reinterpret_cast<float*>(a.scales + i * a.scales_step), a.n_vec, e->unscale[WRITE ? 0 : 1],
                srft_even_start(i + 1, a.shape) - start, block - start};
    } else {
        const int lane = threadIdx.x & 63, first = lane < N ? a.first_block[lane & (N - 1)] : INT32_MAX;
        const int i = (int)__popcll(__ballot(first <= block)) - 1;
        const srft_segment& s = a.seg[i];
        return {s.frag, s.in, s.out, s.scales, s.n_vec, s.unscale, s.blocks, block - __builtin_amdgcn_readlane(first, i)};
    }
}

// ------------------------------------------------------------------------------------------
// read path
// ------------------------------------------------------------------------------------------
// One dword of eight nibbles -> eight exact fp16 codes, as four packed pairs (n_m, n_{m+4}).
// 0x6400 | u is the fp16 number 1024 + u; with u = q + 8, a nibble with its top bit flipped, a packed fp16 subtract of 1032 leaves
// q.  A nibble one position higher (bits 4..7 of the 16-bit half) gives 1024 + 16 u instead; times 1/16 minus 72 is q again
// (exact), which saves the shift.  Selecting the nibble, flipping its bit and setting the exponent is one v_bitop3: nine
// vector-ALU operations per dword (ten with the flip in front).
__device__ __forceinline__ uint32_t and_xor(uint32_t v, uint32_t mask, uint32_t bits) {
    uint32_t r;                                  // (v & mask) ^ bits as one instruction; `bits` is kept in a vector register
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x6a" : "=v"(r) : "v"(v), "s"(mask), "v"(bits));
    return r;
}
__device__ __forceinline__ uint4 decode8(uint32_t v) {
    const half2v bias = {(_Float16)1032.0f, (_Float16)1032.0f};
    const half2v sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f}, bias16 = {(_Float16)72.0f, (_Float16)72.0f};
    const uint32_t low = 0x64086408u, high = 0x64806480u, w = v >> 8;
    uint4 o;
    o.x = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, and_xor(v, 0x000F000Fu, low)) - bias);
    o.y = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, and_xor(v, 0x00F000F0u, high)) * sixteenth - bias16);
    o.z = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, and_xor(w, 0x000F000Fu, low)) - bias);
    o.w = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, and_xor(w, 0x00F000F0u, high)) * sixteenth - bias16);
    return o;
}

// One dword of four two's-complement bytes -> four exact fp16 codes as the packed pairs (b0, b2) and (b1, b3):
// flipping bit 7 gives u = q + 128 in 0..255, 0x6400 | u is 1024 + u, minus 1152 is q.
__device__ __forceinline__ uint2 decode4_bytes(uint32_t v) {
    const half2v bias = {(_Float16)1152.0f, (_Float16)1152.0f};
    const uint32_t bits = 0x64806480u;
    uint2 o;
    o.x = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, and_xor(v, 0x00FF00FFu, bits)) - bias);
    o.y = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, and_xor(v >> 8, 0x00FF00FFu, bits)) - bias);
    return o;
}

// Two fp32 values -> packed fp16, round to nearest even.  The empty asm keeps the compiler from fusing
// the preceding multiply-add into a mixed-precision fma in some copies of this code and not in others:
// every path rounds fp32 -> fp16 the same way, so a vector's output does not depend on where in the
// batch it sits or on the launch shape.
__device__ __forceinline__ uint32_t pack_half2(float a, float b) {
    asm volatile("" : "+v"(a), "+v"(b));
    const half2v h = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(uint32_t, h);
}

// ------------------------------------------------------------------------------------------
// Both kernels are software pipelines over the tiles T_0, T_1, ... of a workgroup (T_k = blockIdx +
// k * gridDim).  Stage k starts with the only barrier of the stage and then, in ONE straight-line
// block, (1) contracts T_k from LDS buffer k % 2 on the matrix cores, (2) runs the vector-ALU tail of
// T_{k-1} (quantizer and stores, or scaling / conversion / stores) on the accumulators the previous
// stage left behind, and (3) moves T_{k+1} from its prefetch registers into LDS buffer (k+1) % 2 and
// refills those registers with T_{k+3}.  (1) and (2) are independent, so one wavefront keeps the MFMA
// pipe and the vector ALU busy together.  The barrier of stage k makes T_k visible and also proves
// that every wavefront has finished reading buffer (k+1) % 2, which (3) overwrites.
//
// The start of a workgroup is the round trip of its loads: T_0 first, then the matrix, then T_1, and T_0 goes to LDS while the
// matrix is on its way.  Against the matrix first and T_0 behind it, us: read 8 plans x 3000 at d = 128 5.1 -> 4.7, 60,000
// vectors 6.6 -> 6.2 (write 7.5 -> 7.3), read 64 x 512 at d = 96 6.0 -> 5.8, 9 x 2000 at d = 224 9.3 -> 8.9; T_1 ahead of
// the matrix as well: 4.7, 6.6 (7.9), 6.0, 9.1.
//
// Rows past the end of the input alias to the last row, in the loads AND in the stores: surplus lanes
// compute the last vector again and store the same bytes to the same place.  Prefetches past the last
// tile re-read the last tile.  So no memory operation in the loop is conditional, the hardware wait
// counters are exact, and stores and younger prefetches stay in flight while older data is consumed.
// Every branch in the kernels is uniform over the workgroup.
// ------------------------------------------------------------------------------------------

// Running maximum of non-negative floats kept as their bit patterns (they order alike).  All workgroups of a launch
// update the same few cache lines at about the same time, and atomics to one line are served one after the other:
// the current value is read first (from L2, past the caches of this compute unit), and the atomic is only sent when
// it would raise it -- of N similar contributions about ln N do.
__device__ __forceinline__ void atomic_max_nonneg(unsigned int* p, float v) {
    const unsigned int bits = __float_as_uint(v);
    if (bits > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(p, bits);
}

// End of a workgroup's share of the abs-max statistic: `part` (LDS) holds 32 rows of D channel maxima, kAmaxRow floats
// apart; thread c < D takes the maximum of channel c and updates amax[c].  A wavefront thus sends one request of 64
// neighbouring channels where a lane per channel and half used to send 2 channels a request: on a statistic that starts at
// zero every workgroup's request is sent (they all end together), and a launch over 1,000,003 vectors at d = 128 spent
// 190 of its 231 us in them.
template <int D> constexpr int kAmaxRow = D + 4;         // padded: the lanes that write a column hit different banks
// SUB teams of threads each bring 32 rows, team_floats apart, and add up their own before the first team updates amax.
template <int D, int SUB = 1>
__device__ __forceinline__ void publish_amax(float* part, size_t team_floats, unsigned int* amax, float unscale) {
    const int team = SUB > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / (blockDim.x / SUB)) : 0;
    const int c = threadIdx.x - team * (blockDim.x / SUB);
    float* const mine = part + team * team_floats;
    __syncthreads();
    float m = 0.0f;
    if (c < D) {
        m = mine[c];
#pragma unroll
        for (int r = 1; r < kTileVecs; ++r) m = fmaxf(m, mine[r * kAmaxRow<D> + c]);
        if constexpr (SUB > 1) mine[c] = m;                  // (row 0 of this channel: nobody else reads it)
    }
    if constexpr (SUB > 1) {
        __syncthreads();
        if (team > 0) return;
#pragma unroll
        for (int k = 1; k < SUB; ++k) m = fmaxf(m, part[k * team_floats + (c < D ? c : 0)]);
    }
    if (c < D) atomic_max_nonneg(&amax[c], m * unscale);
}

// Where the input rows of the write path lie.  srft_rows_dense: one after the other from x on.
struct srft_rows_dense {};
// srft_rows_paged: the rows of a cache's pages that a flush converts (cache_flush.h).  Row v is slot v % R of sequence v / R %
// n_seq of page v / (n_seq R), token j = page R + slot of its sequence counted from the first page on; the first `held` tokens of
// a sequence are in the view already, in the place of row v, the others are where the caller has them, [n_seq][t_all][U units].
// Row and unit numbers are 32-bit, and the divisions exact, by the host's check (srft_flush_fits).
struct srft_rows_paged {
    const uint4 *fresh, *view;
    int page_rows, R, held, t_all;
    uint32_t page_magic, slot_magic;
    template <int U>
    __device__ __forceinline__ const uint4* row(int v) const {
        const int page = srft_even_segment((uint32_t)v, page_magic), in_page = v - page * page_rows;
        const int seq = srft_even_segment((uint32_t)in_page, slot_magic), j = page * R + in_page - seq * R;
        return j < held ? view + (unsigned)(v * U) : fresh + (unsigned)((seq * t_all + j - held) * U);
    }
};

// Which tiles a workgroup of a per-plan launch walks: first tile, stride, and the end (exclusive) of its range.
__device__ __forceinline__ bool srft_tile_range(long long n_vec, int& t0, int& stride, int& t_end) {
    t0 = blockIdx.x;
    stride = gridDim.x;
    t_end = (int)((n_vec + kTileVecs - 1) / kTileVecs);
    return t0 < t_end;
}

#endif  // SRFT_DEVICE_UTIL_H
