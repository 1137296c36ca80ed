// common.h -- shared declarations of the fused SRFT int4 KV-cache quantizer / dequantizer for MI355X (gfx950).
//
// How the path is mapped to CDNA4
// -------------------------------
// Per vector the method is: sign flip, unitary real DFT with the real packing of Eq. 2, per-channel
// lambda, per-group abs-max, round to int4, nibble pack (Sec. 3.2, Sec. 5.1, Sec. 7.1).  Sign, DFT,
// packing and lambda are all linear, so together they are ONE real d x d matrix
//     W = diag(lambda) * Q * diag(s),        Q = pack o F   (orthogonal),
// and the read path is the matrix  R = diag(s) * Q^T * diag(1 / max(lambda, 1e-6)).
// At 5.6 TB/s a d = 128 vector has about 37 compute-unit clocks; a butterfly FFT plus the fp16
// conversions needs about 3000 vector-ALU lane operations per vector, more than the 64 lanes x 37
// clocks available, whereas the matrix cores do the dense product with time to spare.  So the
// transform runs on MFMA (v_mfma_f32_32x32x16_f16) and the vector ALU only does the quantizer.
//
// Exactness: x is fp16, hence an exact MFMA operand.  W is split on the host into two fp16
// matrices W = Whi + Wlo (after a power-of-two scaling that keeps Wlo out of the fp16 denormal
// range); both products accumulate into the same fp32 accumulator, which gives about 22 bits of W.
// On the read path the codes (integers in [-8, 7]) are exact fp16 operands; the per-(vector, group)
// scale cannot enter the matrix, so each group's 32 codes are contracted separately (K = 32) and
// the partial results are combined as  x = sum_j scale_j * P_j  on the vector ALU in fp32.
//
// Work decomposition (plain forms): a workgroup has d/32 wavefronts and walks over tiles of 32 vectors
// (persistent grid).  Wavefront w owns the 32 output rows 32w..32w+31 -- on the write path that is
// exactly quantization group w, so the abs-max needs a single cross-lane step -- and keeps its
// 32 x d slab of the matrix (hi and lo) in registers for the whole launch.  The 32 x d operand tile
// (inputs, or decoded codes) is loaded once per workgroup with coalesced 16-byte accesses, staged in
// LDS (double buffered, one barrier per tile, reached by every thread) and read by every wavefront.
// The MFMA row order inside a slab is permuted on the host so that a lane ends up holding 16
// CONSECUTIVE outputs: 16 nibbles = one 8-byte store on the write path, 16 fp16 = two 16-byte
// stores on the read path, with no cross-lane shuffles.
//
// Folded forms (d = 128 and 256 on the write path, 128 / 192 / 256 on the read path): symmetries of Q let
// outputs share half-length (folded once) or quarter-length (folded twice) partial sums, which halves or
// quarters the matrix work; they are described at srft_quantize_fold_tiles, in quantize_fold4_tiles.h, at
// the FOLD parameter of srft_dequantize_tiles and in dequantize_fold4_tiles.h.
//
// Around the two paths: the same kernels serving several plans in one launch (a segment table passed as a
// kernel argument), the per-channel abs-max statistic lambda is calibrated from, an 8-bit code width, the
// Walsh-Hadamard matrix in place of the DFT (the comparator of Sec. 3.1), scores of queries against the stored
// record without reconstructing the keys, and a host-side cache manager (int4 store, fp16 residual window,
// dequantized view) built on the batched launches.
//
// The kernels run at the socket's power limit with a throttled clock, so what shortens them is work per vector
// (matrix instructions, vector instructions, LDS traffic), not more parallelism: see the folded forms.
//
// Source layout: the kernel templates live in quantize_tiles.h (write path, plain form), quantize_fold_tiles.h and
// quantize_fold4_tiles.h (write path, folded forms), dequantize_tiles.h and dequantize_fold4_tiles.h (read path),
// kernels/scores.hip, kernels/attend.hip and kernels/decode_attention.hip; every file under kernels/
// instantiates one family of them and exports a function that picks the instance for a plan; plan.hip builds
// the constant tables, api.hip holds the C entry points, cache.hip the cache manager.
#ifndef SRFT_COMMON_H
#define SRFT_COMMON_H

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <vector>

#include "launch_shape.h"
#include "srft_kv.h"

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));   // scales and scores are 4-byte aligned
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kTileVecs = 32;          // vectors per tile = N of the 32x32x16 MFMA
constexpr int kMaxD = 256;
constexpr int kMaxAttendStripes = 2048;      // value-side kernel: most workgroups per channel slab (each owns 32 x d floats of workspace)
constexpr int kAttendFan = 64;                // value-side kernel: first-level sums the partial results are added into
constexpr float kMinScale = 7.888609052210118e-31f;   // 2^-100: below this a group is stored as zero
// The kernels index tiles of 32 vectors with 32-bit integers and look a few grid strides ahead.
constexpr int64_t kMaxVectors = (int64_t)1 << 33;

// group mode of a plan.  kGroup32: one scale per slab (g = 32, the deployed format).  kGroup16: one scale per
// lane (g = 16).  kGroupWide: g = 32 * gw with gw >= 2 slabs per group, up to the per-token case g = d.
enum { kGroup16 = 0, kGroup32 = 1, kGroupWide = 2 };
// what the write-path kernel produces (see quantize_tiles.h)
enum { kOutCodes = 0, kOutRaw = 1, kOutAmax = 2 };

// Several plans in one launch (a decode step appends a few hundred vectors to each of many (layer, K|V)
// caches: one launch per plan would be all launch latency).  A segment = a plan's constants and buffers, or a part of them
// (launch_shape.h); it is served by workgroups first_block[i] .. first_block[i] + seg[i].blocks - 1, each walking that
// segment's tiles with that many as stride.  Entries of first_block past the last segment hold INT32_MAX.  The table travels
// as a kernel argument.
constexpr int kMaxBatch = 64;       // the table is about 3.8 KiB of the 4 KiB a kernel may take as arguments
// Up to kFewBatch segments travel in a table of their own: the runtime writes the arguments of a launch out one by one, 0.8 us
// of a launch's 4 us for 3.8 KiB (append of 2 x 256 vectors at d = 128: 5.9 -> 5.4 us a call).
constexpr int kFewBatch = 8;
struct srft_segment {
    const uint4* frag;
    const void* in;                 // write path: x      read path: codes
    void* out;                      // write path: codes  read path: out
    float* scales;                  // written / read
    long long n_vec;
    float unscale;
    int blocks;
};
template <int N>
struct srft_batch {
    int first_block[N];
    srft_segment seg[N];
};
// What the kernels need of a plan, per path (0 = write, 1 = read): an entry of the device's plan table (plan.hip).
struct srft_plan_entry {
    uint64_t table[2];                                        // device addresses
    float unscale[2];
    uint64_t unused;
};
// Segments of one length whose addresses (and whose plans' entries) lie a constant number of bytes apart: a cache that is one
// tensor over its layers, a step that appends the same number of vectors to each.  A launch of up
// to 104 bytes of arguments takes 2.7-2.9 us of the host, one of 112 to 900 3.5, one of 3.8 KiB 4.2, and any number of segments
// fits.  us a call, against the tables: write 2 plans x 256 vectors at d = 128 4.1 -> 3.8, 64 x 512 at d = 96 4.9 -> 4.3,
// 100 x 700 at d = 128 13.7 -> 8.9 (two launches before), read 9 x 100 at d = 96 5.3 -> 4.6; 56 x 8192 and 4 x 1,048,576
// within 0.5 %.
// The entry is one more load in front of the matrix.  With a gigabyte of other traffic before every call: write 64 x 512 at
// d = 96 10.6 -> 10.2, 2 x 256 at d = 128 6.4 and 6.4, read 9 x 100 at d = 96 6.8 -> 6.4, 56 x 16 at d = 128 7.1 -> 6.7;
// over 48, 300, 150 and 48 sets of plans and buffers in turn 6.65 -> 6.2, 3.6 and 3.6, 3.85 -> 3.5, 4.2 -> 3.65.
template <>
struct srft_batch<0> {
    const srft_plan_entry* plan;
    const char* in;
    char* out;
    char* scales;
    long long plan_step, in_step, out_step, scales_step;      // bytes
    long long n_vec;                                          // of each segment
    srft_even_shape shape;                                    // which workgroups serve which
};
using srft_batch_even = srft_batch<0>;
static_assert(sizeof(srft_batch_even) + sizeof(int) <= 96, "a small launch");
using srft_batch_many = srft_batch<kMaxBatch>;
using srft_batch_few = srft_batch<kFewBatch>;
static_assert(sizeof(srft_batch_many) + sizeof(int) <= 4096, "kernel arguments are limited to 4 KiB");

// A cache's pages that became full, over all its plans (cache_flush.h): buffers and plan entries lie a constant step apart, as in
// srft_batch_even.  codes, scales and view start at the first of these pages, fresh at the new tokens.
struct srft_flush {
    const srft_plan_entry* plan;
    const char* fresh;
    char *view, *codes, *scales;
    long long plan_step, fresh_step, view_step, codes_step, scales_step;      // bytes
    srft_even_shape shape;
    int n_vec;                              // of each plan
    int page_rows, R, held, t_all, tail;    // rows of a page (n_seq R); tokens a sequence's window holds, brings, and keeps
    uint32_t page_magic, slot_magic;        // division by page_rows and R
    int gw;
};
struct flush_kernels_t {
    typedef void (*kernel)(const srft_flush);
    kernel write, whole;                    // without and with the read path (null at d = 160, 192, 224 and plain d = 256: not built)
    flush_kernels_t(std::nullptr_t = nullptr) : write(nullptr), whole(nullptr) {}
    flush_kernels_t(kernel w, kernel all) : write(w), whole(all) {}
};

typedef void (*quantize_kernel_t)(const uint4*, const uint4*, long long, uint2*, float*, float4*, float, float, int);
typedef void (*dequantize_kernel_t)(const uint4*, const uint2*, const float*, long long, uint4*, float, int);
struct batched_kernels_t {
    void (*many)(const srft_batch_many, int);
    void (*few)(const srft_batch_few, int);
    void (*even)(const srft_batch_even, int);
    batched_kernels_t(std::nullptr_t = nullptr) : many(nullptr), few(nullptr), even(nullptr) {}
    batched_kernels_t(void (*m)(const srft_batch_many, int), void (*f)(const srft_batch_few, int), void (*e)(const srft_batch_even, int))
        : many(m), few(f), even(e) {}
};
#define SRFT_BATCHED(kernel, ...) batched_kernels_t(kernel<__VA_ARGS__, kMaxBatch>, kernel<__VA_ARGS__, kFewBatch>, kernel<__VA_ARGS__, 0>)

struct srft_plan {
    int d = 0, g = 0, bits = 4, transform = 0, device = 0;
    uint64_t seed = 0;
    std::vector<int8_t> signs;
    char* memory = nullptr;     // the allocation that holds the tables below (device)
    uint4* wfrag = nullptr;     // write-path matrix fragments (device)
    uint4* rfrag = nullptr;     // read-path matrix fragments (device)
    uint4* rfold = nullptr;     // read-path fragments of the folded form (device), when fold_dq
    uint4* wfold = nullptr;     // write-path fragments of the folded form (device), when fold_q
    uint4* wfold4 = nullptr;    // write-path table of the twice-folded form (device): d = 256, DFT
    uint4* rfold4 = nullptr;    // read-path table of the twice-folded form (device), when fold4_dq
    float* rmat_f32 = nullptr;  // R^T in fp32, [k][n] = s_n Q[k][n] / max(lambda_k, 1e-6) (device): the one inverse transform per
                                // query of srft_kv_attend
    int compute_units = 0;
    float* bfly = nullptr;      // table of the butterfly form of the write path (device), d = 128 or 256 / g = 32 / 4-bit only
    float* q_table = nullptr;   // table of the queries' transform (device; rotated_queries.h), d a multiple of 64
    bool fold_dq = false;       // read path contracts even and odd codes separately (half the matrix work)
    bool fold_q = false;        // write path contracts even and odd inputs separately (half the matrix work)
    bool fold4_q = false;       // write path contracts the inputs in four classes n mod 4 (a quarter of the work)
    bool fold4_dq = false;      // read path contracts (cosine | sine) x (even | odd) codes apart (a quarter of the work)
    float unscale_w = 1.0f;     // 2^-e of the write matrix
    float unscale_r = 1.0f;
    float unscale_r4 = 1.0f;    // 2^-e of the twice-folded read table
    int grid_q = 0, grid_dq = 0;    // default persistent grid sizes
    int grid_staged = 0;            // ... of the write path's plain form with the record through LDS (elsewhere grid_q)
    int grid_flush = 0;             // ... of a cache's flush with both paths in one launch (0: there is no such kernel)
    int slabs_q = 1, slabs_dq = 1;  // slabs of the matrix per wavefront in the write / read kernel
    int gm = 1, gw = 1;             // group mode (kGroup16 / kGroup32 / kGroupWide) and slabs per group
    int max_wgs = 0;
    srft_plan_entry* entry = nullptr;   // this plan's entry in the device's plan table (device; null where the table is full)
};

struct srft_cache {
    std::vector<const srft_plan*> plans;
    std::vector<uint8_t*> codes;
    std::vector<float*> scales;
    std::vector<void*> view;
    int n_seq = 0, R = 0;
    int64_t capacity = 0, tokens = 0, quantized = 0;
};

// ---- kernel instances, one function per translation unit under kernels/ (nullptr: no such instance) ----
// write path, plain form, codes out: d, group mode, way of the record (srft_write_staged); 4- and 8-bit codes.
quantize_kernel_t srft_pick_quantize_plain_b4(int d, int gm, bool staged);
quantize_kernel_t srft_pick_quantize_plain_b8(int d, int gm, bool staged);
batched_kernels_t srft_pick_quantize_plain_batched_b4(int d, int gm, bool staged);
batched_kernels_t srft_pick_quantize_plain_batched_b8(int d, int gm, bool staged);
// write path, plain form, other outputs (kOutRaw, kOutAmax)
quantize_kernel_t srft_pick_quantize_aux(int d, int slabs, int out, int teams);
// write path, folded form (d = 128, 256)
quantize_kernel_t srft_pick_quantize_fold(int d, int bits, bool wide, bool through);
// Teams of wavefronts per workgroup of the abs-max statistic, by head dimension, form of the write path (0 plain, 1 once, 2
// twice folded) and tiles.  Teams leave fewer workgroups, up to one per compute unit, that update the statistic's cache lines one
// after the other; but they start later (each with its matrix), share their barriers, and a call of few tiles wants them on
// different compute units.  So: one team up to a few hundred tiles, teams from there on, and one team again where the rate counts
// and not the end.  us, one team -> the teams of this rule, a statistic that has its values / one that starts at zero (cleared by
// a kernel in front, 2.3 us):
//   d = 32   8,000 vectors 2.5 / 5.4 (eight teams: 2.7 / 5.3)   24,000 3.0 / 6.4 -> 2.8 / 5.8   1,000,003 13.4 / 25.4 -> 11.9 / 15.7
//   d = 64   3,000 2.5 / 5.4 (four: 3.1 / 5.7)   8,000 3.5 / 7.1 -> 3.1 / 6.3   1,000,003 23.1 / 41.6 -> 23.5 / 28.9 (eight: 24.9 /
//            29.3)   8,000,000 166 / 186 (four: 189 / 191, eight: 177 / 174)
//   d = 96   60,000 5.5 / 10.8 (four: 6.6 / 13.4)   400,000 14.7 / 24.2 (15.9 / 22.0)   1,000,003 39.5 / 51.4 -> 41.2 / 42.8
//            4,000,000 164 / 167 -> 137 / 139
//   d = 128  plain: 60,000 6.6 / 12.0 (two: 7.4 / 13.8)   200,000 13.5 / 18.5 -> 13.1 / 19.3   524,288 35.1 / 43.1 -> 32.9 / 37.6
//            2,000,000 107 / 117 (two: 115 / 118)
//   d = 128  folded: 3,000 3.1 / 6.1 (two: 3.9 / 6.7)   8,000 4.6 / 8.4 -> 4.3 / 7.9 (four: 5.7 / 8.8)   100,000 12.7 / 19.2 -> 9.6 /
//            15.9 (four: 10.3 / 18.1)   1,000,003 49.9 / 61.8 -> 50.3 / 54.0 (two: 60.8 / 64.1)   3,000,000 132 / 141 (four: 137 / 140)
//   d = 256  8,000 6.5 / 10.4 (two: 6.8 / 9.9)   24,000 9.2 / 14.2 -> 9.7 / 13.0   300,000 43.0 / 48.5 -> 37.5 / 44.4
//            1,000,003 146 / 148 -> 120 / 123
constexpr int srft_amax_teams(int d, int form, long long tiles) {
    if (form == 2) return tiles < 512 ? 1 : 2;
    if (form == 1) return tiles < 200 || tiles >= 65536 ? 1 : tiles < 8192 ? 2 : 4;
    if (d == 32) return tiles < 400 ? 1 : 8;
    if (d == 64) return tiles < 200 || tiles >= 131072 ? 1 : 4;
    if (d == 96) return tiles < 16384 ? 1 : 4;
    if (d == 128) return tiles < 2560 || tiles >= 32768 ? 1 : 2;
    return 1;
}
quantize_kernel_t srft_pick_quantize_fold_amax(int teams);  // the abs-max statistic through the once-folded contraction (d = 128)
batched_kernels_t srft_pick_quantize_fold_batched(int d, int bits, bool wide, bool through);
// write path, folded twice (d = 256; g = 16, 32 and 256); the abs-max statistic; the size of its table in 16-byte units
quantize_kernel_t srft_pick_quantize_fold4(int bits, int gm);
quantize_kernel_t srft_pick_quantize_fold4_amax(int teams);
batched_kernels_t srft_pick_quantize_fold4_batched(int bits, int gm);
int srft_fold4_table_units(void);
// read path (through: the rows are written through to memory, srft_read_through)
dequantize_kernel_t srft_pick_dequantize_b4(int d, int slabs, int gm, bool through);
dequantize_kernel_t srft_pick_dequantize_b8(int d, int slabs, int gm, bool through);
batched_kernels_t srft_pick_dequantize_batched_b4(int d, int slabs, int gm, bool through);
batched_kernels_t srft_pick_dequantize_batched_b8(int d, int slabs, int gm, bool through);
// read path, folded twice (d = 128 at g >= 32, d = 256; fine: g = 16); the size of its table in 16-byte units
dequantize_kernel_t srft_pick_dequantize_fold4(int d, int bits, bool fine, bool through);
batched_kernels_t srft_pick_dequantize_fold4_batched(int d, int bits, bool fine, bool through);
int srft_rfold4_table_units(int d);
// a cache's flush (cache_flush.h)
flush_kernels_t srft_pick_cache_flush_plain(int d, int bits, int gm, bool staged);
flush_kernels_t srft_pick_cache_flush_fold(int d, int bits, int gm, bool fold4_q);
flush_kernels_t srft_plan_flush_kernels(const srft_plan* p, int* threads, bool staged = false);
// write path with the transform as FFT butterflies on the vector ALU (d = 128 or 256, g = 32, 4-bit; the comparison form)
int srft_launch_quantize_butterfly(int d, const float* table_dev, const void* x, long long n_vec, uint8_t* codes,
                                   float* scales, int max_workgroups, hipStream_t st);
// scores in the rotated domain (kernels/scores.hip)
int srft_launch_scores(const srft_plan* p, const void* q, int n_q, const uint8_t* codes, const float* scales,
                       long long n_keys, float* out, hipStream_t st);

// weighted sums of the stored values in the rotated domain (kernels/attend.hip): workgroups per channel slab for
// n_q queries over n_keys values, and the three launches (partial sums per workgroup into `part`, their fixed-order
// reduction, the inverse transform)
int srft_attend_stripes(const srft_plan* p, int n_q, long long n_keys);
// workspace: part [kMaxAttendStripes][32][d], part2 [kAttendFan][32][d] (and room of another 32 floats each, which callers'
// buffers have always had)
constexpr size_t srft_attend_workspace_floats(int d) { return (size_t)(kMaxAttendStripes + kAttendFan) * 32 * (d + 1); }
int srft_launch_attend(const srft_plan* p, const float* w, int n_q, const uint8_t* codes, const float* scales,
                       long long n_keys, float* out, float* part, hipStream_t st);

// one decode step of attention in one pass over both records (kernels/decode_attention.hip)
int srft_launch_decode_attention(const srft_plan* pk, const srft_plan* pv, const void* q, int n_q, const uint8_t* k_codes,
                                 const float* k_scales, const uint8_t* v_codes, const float* v_scales, long long n_keys,
                                 float softmax_scale, float* out, void* workspace, hipStream_t st);

// ---- host side (plan.hip, api.hip) ----
int srft_hip_fail(hipError_t e);         // records the error for srft_last_hip_error, returns SRFT_ERR_HIP
#define SRFT_HIP(call)                                   \
    do {                                                 \
        hipError_t e_ = (call);                          \
        if (e_ != hipSuccess) return srft_hip_fail(e_);  \
    } while (0)

// The body of an entry point that allocates on the host: what it throws becomes a status.
template <class F>
int srft_no_throw(F body) {
    try {
        return body();
    } catch (...) {
        return srft_hip_fail(hipErrorOutOfMemory);
    }
}

// One launch.  (The triple-chevron form and hipLaunchKernelGGL park the configuration and fetch it back, 0.1-0.2 us.)
// A refusal is told once, by the return value: HIP's last error, which the caller's own checks read, is cleared.
template <class T> struct srft_same { using type = T; };
template <class... P>
int srft_launch(void (*kernel)(P...), dim3 grid, int threads, hipStream_t st, const typename srft_same<P>::type&... args) {
    void* p[] = {const_cast<void*>(static_cast<const void*>(&args))...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3((unsigned)threads), p, 0, st);
    if (e == hipSuccess) return SRFT_OK;
    (void)hipGetLastError();
    return srft_hip_fail(e);
}

// the kernels a plan launches, and their block sizes
// (tiles: of the launch; lines: its results start at a multiple of 64 bytes)
quantize_kernel_t srft_plan_quantize_kernel(const srft_plan* p, int out, int* threads, long long n_tiles = 0, bool lines = true);
dequantize_kernel_t srft_plan_dequantize_kernel(const srft_plan* p, int* threads, long long n_tiles = 0, bool lines = true);
// the tables and the matrix scaling the kernels of a plan take
inline int srft_plan_amax_teams(const srft_plan* p, long long n_tiles) {
    return srft_amax_teams(p->d, p->wfold4 ? 2 : p->fold_q ? 1 : 0, n_tiles);
}
// the bytes of this many tiles, fp16 vectors and record
inline long long srft_plan_bytes(const srft_plan* p, long long tiles) {
    return tiles * kTileVecs * (2LL * p->d + p->d * p->bits / 8 + 4 * (p->d / p->g));
}
inline bool srft_plan_fold_through(const srft_plan* p, long long tiles, bool lines) {
    return srft_fold_through(p->d, p->bits, lines, srft_plan_bytes(p, tiles));
}
inline bool srft_plan_read_through(const srft_plan* p, long long tiles, bool lines) {
    return srft_read_through(p->d, lines, srft_plan_bytes(p, tiles));
}
// the way of the record of a launch of the write path's plain form over this many tiles, and the most workgroups of a launch
inline bool srft_plan_staged(const srft_plan* p, long long tiles, bool lines) {
    return !p->fold_q && !p->fold4_q && srft_write_staged(p->d, p->g, p->bits, lines, tiles, p->max_wgs > 0 ? p->max_wgs : p->grid_q, p->compute_units);
}
inline long long srft_plan_write_grid(const srft_plan* p, long long tiles, bool lines) {
    return p->max_wgs > 0 ? p->max_wgs : srft_plan_staged(p, tiles, lines) ? p->grid_staged : p->grid_q;
}
inline const uint4* srft_plan_write_table(const srft_plan* p) { return p->fold4_q ? p->wfold4 : p->fold_q ? p->wfold : p->wfrag; }
inline const uint4* srft_plan_read_table(const srft_plan* p) { return p->fold4_dq ? p->rfold4 : p->fold_dq ? p->rfold : p->rfrag; }
inline float srft_plan_read_unscale(const srft_plan* p) { return p->fold4_dq ? p->unscale_r4 : p->unscale_r; }
// batched launches over plans that share shape and kernel choice (api.hip)
int srft_run_batched(const srft_plan_t* const* plans, const void* const* in0, const void* const* in1,
                     void* const* out0, void* const* out1, const int64_t* n_vec, int count, bool write_path,
                     hipStream_t st);
// true when two plans can share one batched launch or one cache (shape, code width, transform, device, kernel forms)
bool srft_plans_compatible(const srft_plan* a, const srft_plan* b);

inline bool srft_aligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

#define SRFT_DISPATCH_D(d, fn, ...)                       \
    switch (d) {                                          \
        case 32:  return fn<32>(__VA_ARGS__);             \
        case 64:  return fn<64>(__VA_ARGS__);             \
        case 96:  return fn<96>(__VA_ARGS__);             \
        case 128: return fn<128>(__VA_ARGS__);            \
        case 160: return fn<160>(__VA_ARGS__);            \
        case 192: return fn<192>(__VA_ARGS__);            \
        case 224: return fn<224>(__VA_ARGS__);            \
        case 256: return fn<256>(__VA_ARGS__);            \
        default:  return nullptr;                         \
    }

#endif  // SRFT_COMMON_H
