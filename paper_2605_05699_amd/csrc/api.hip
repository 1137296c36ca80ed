// api.hip -- the C entry points of the write path, the read path and what sits around them: argument checks
// (all before the first HIP call), grid sizing, launches.
#include <algorithm>
#include <cmath>
#include <numeric>

#include "common.h"
#include "launch_shape.h"

namespace {

// Workgroups of the abs-max statistic.  Each ends with one request per 32 channels to the same few cache lines, served one
// after the other (about 11 ns a workgroup at d = 128, all at once at the end), so more workgroups shorten the streaming
// and lengthen the end: the sum is smallest near sqrt(tiles) times a constant.  At most what reaches the read rate: with teams
// (srft_amax_teams) and where one team is five wavefronts or more (d >= 160) one per compute unit, two with three wavefronts
// (d = 96), with one to four wavefronts what the write path's grid holds.  us for 100,000 / 200,000 / 300,000 vectors at d = 192, up
// to one per unit against up to two: 15.5 / 27.7 / 43.5 and 25.0 / 33.8 / 48.9.
long long amax_grid(const srft_plan* p, long long n_tiles, int teams) {
    const long long cus = p->compute_units, most = teams > 1 || p->d >= 160 ? cus : p->d == 96 ? 2 * cus : p->grid_q;
    return std::min((long long)(5.0 * std::sqrt((double)n_tiles)) + 1, most);
}

int launch_quantize(const srft_plan* p, const void* x, long long n, uint8_t* codes, float* scales, float* wout,
                    int out, hipStream_t st) {
    const long long n_tiles = (n + kTileVecs - 1) / kTileVecs;
    const int teams = out == kOutAmax ? srft_plan_amax_teams(p, n_tiles) : 1;
    const bool lines = srft_aligned(codes, 64);
    long long grid = out == kOutCodes ? srft_plan_write_grid(p, n_tiles, lines)
                     : p->max_wgs > 0 ? p->max_wgs
                     : out == kOutAmax ? amax_grid(p, n_tiles, teams)
                                       : p->grid_q;
    grid = std::min(grid, (n_tiles + teams - 1) / teams);    // no workgroup without a tile
    int threads = 0;
    const quantize_kernel_t kernel = srft_plan_quantize_kernel(p, out, &threads, n_tiles, lines);
    if (!kernel) return SRFT_ERR_BAD_D;
    const bool fold4 = out == kOutCodes ? p->fold4_q : out == kOutAmax && p->wfold4;
    const bool fold = p->fold_q && (out == kOutCodes || out == kOutAmax);
    // the twice-folded form carries the matrix scaling inside its per-channel factors
    const float unscale = fold4 ? 1.0f : p->unscale_w;
    return srft_launch(kernel, dim3((unsigned)grid), threads, st, fold4 ? p->wfold4 : fold ? p->wfold : p->wfrag, (const uint4*)x,
                       n, (uint2*)codes, scales, (float4*)wout, unscale, unscale / (p->bits == 8 ? 127.0f : 7.0f), p->gw);
}

int launch_dequantize(const srft_plan* p, const uint8_t* codes, const float* scales, long long n, void* out,
                      hipStream_t st) {
    const long long n_tiles = (n + kTileVecs - 1) / kTileVecs;
    long long grid = p->max_wgs > 0 ? p->max_wgs : p->grid_dq;
    if (grid > n_tiles) grid = n_tiles;
    int threads = 0;
    const dequantize_kernel_t kernel = srft_plan_dequantize_kernel(p, &threads, n_tiles, srft_aligned(out, 64));
    if (!kernel) return SRFT_ERR_BAD_D;
    return srft_launch(kernel, dim3((unsigned)grid), threads, st, srft_plan_read_table(p), (const uint2*)codes, scales, n,
                       (uint4*)out, srft_plan_read_unscale(p), p->gw);
}

// The part of a segment that a share walks.
srft_segment segment_part(const srft_plan* p, bool write_path, const srft_segment& whole, const srft_share& sh) {
    const long long code_bytes = (long long)p->d * p->bits / 8, row_bytes = 2LL * p->d, v0 = sh.tile * kTileVecs;
    srft_segment s = whole;
    s.in = (const char*)s.in + v0 * (write_path ? row_bytes : code_bytes);
    s.out = (char*)s.out + v0 * (write_path ? code_bytes : row_bytes);
    s.scales += v0 * (p->d / p->g);
    s.n_vec = std::min(s.n_vec - v0, sh.tiles * kTileVecs);
    return s;
}

// The kernels of a plan's batched launches, and their block size.  tiles: of the launch; lines: its results start at multiples of 64
// bytes.
batched_kernels_t batched_kernels(const srft_plan* p, bool write_path, long long tiles, bool lines, int* threads) {
    if (write_path && p->fold4_q) {
        *threads = 256;
        return srft_pick_quantize_fold4_batched(p->bits, p->gm);
    }
    if (write_path && p->fold_q) {
        *threads = p->d;
        return srft_pick_quantize_fold_batched(p->d, p->bits, p->gm == kGroupWide, srft_plan_fold_through(p, tiles, lines));
    }
    if (write_path) {
        *threads = 2 * p->d / p->slabs_q;
        const bool staged = srft_plan_staged(p, tiles, lines);
        return p->bits == 8 ? srft_pick_quantize_plain_batched_b8(p->d, p->gm, staged) : srft_pick_quantize_plain_batched_b4(p->d, p->gm, staged);
    }
    const bool through = srft_plan_read_through(p, tiles, lines);
    if (p->fold4_dq) {
        *threads = p->d;
        return srft_pick_dequantize_fold4_batched(p->d, p->bits, p->gm == kGroup16, through);
    }
    *threads = 2 * p->d / p->slabs_dq;
    return p->bits == 8 ? srft_pick_dequantize_batched_b8(p->d, p->slabs_dq, p->gm, through)
                        : srft_pick_dequantize_batched_b4(p->d, p->slabs_dq, p->gm, through);
}

// One batched launch over the first `count` segments of the table, which is complete except for the workgroups.
int launch_batched(const srft_plan* p, srft_batch_many& whole, int count, bool write_path, bool lines, hipStream_t st) {
    long long tiles[kMaxBatch];
    for (int i = 0; i < count; ++i) tiles[i] = (whole.seg[i].n_vec + kTileVecs - 1) / kTileVecs;
    srft_share shares[kMaxBatch];
    int next = 0;
    const long long all = std::accumulate(tiles, tiles + count, 0LL);
    const long long budget = write_path ? srft_plan_write_grid(p, all, lines) : p->max_wgs > 0 ? p->max_wgs : p->grid_dq;
    const int n = srft_share_out(tiles, count, budget, shares, kMaxBatch, &next);
    srft_batch_many cut;
    if (n > count)
        for (int i = 0; i < n; ++i) cut.seg[i] = segment_part(p, write_path, whole.seg[shares[i].segment], shares[i]);
    srft_batch_many& a = n > count ? cut : whole;
    for (int i = 0; i < n; ++i) {
        a.first_block[i] = shares[i].first_block;
        a.seg[i].blocks = shares[i].blocks;
    }
    for (int i = n; i < kMaxBatch; ++i) a.first_block[i] = INT32_MAX;
    int threads = 0;
    const batched_kernels_t kernel = batched_kernels(p, write_path, all, lines, &threads);
    if (!kernel.many) return SRFT_ERR_BAD_D;
    if (n <= kFewBatch) {
        srft_batch_few few;
        std::copy_n(a.first_block, kFewBatch, few.first_block);
        std::copy_n(a.seg, n, few.seg);
        return srft_launch(kernel.few, dim3((unsigned)next), threads, st, few, p->gw);
    }
    return srft_launch(kernel.many, dim3((unsigned)next), threads, st, a, p->gw);
}

// The whole batch as one launch without a table, where its counts are equal and its addresses and plan entries a constant step
// apart (srft_batch_even).  False: not such a batch.
bool even_batch(const srft_plan_t* const* plans, const void* const* in, void* const* out, const void* const* scales,
                const int64_t* n_vec, int count, bool write_path, bool lines, srft_batch_even* a) {
    for (int i = 1; i < count; ++i)
        if (n_vec[i] != n_vec[0]) return false;
    if (n_vec[0] == 0 || !plans[0]->entry) return false;
    a->plan_step = count > 1 ? (long long)((uintptr_t)plans[1]->entry - (uintptr_t)plans[0]->entry) : 0;
    for (int i = 1; i < count; ++i)
        if (!plans[i]->entry || (uintptr_t)plans[i]->entry - (uintptr_t)plans[i - 1]->entry != (uintptr_t)a->plan_step) return false;
    if (!srft_even_step(in, count, &a->in_step) || !srft_even_step(out, count, &a->out_step) ||
        !srft_even_step(scales, count, &a->scales_step))
        return false;
    const srft_plan* p = plans[0];
    const long long tiles = (n_vec[0] + kTileVecs - 1) / kTileVecs;
    const long long budget = write_path ? srft_plan_write_grid(p, tiles * count, lines) : p->max_wgs > 0 ? p->max_wgs : p->grid_dq;
    const int blocks = srft_even_blocks(tiles, count, budget);
    if (blocks == 0) return false;
    a->shape = srft_even_spread(tiles, count, write_path ? (long long)blocks * count : budget, blocks);
    a->plan = p->entry;
    a->in = (const char*)in[0];
    a->out = (char*)out[0];
    a->scales = (char*)scales[0];
    a->n_vec = n_vec[0];
    return true;
}

}  // namespace

// Shared body of the two batched entry points.  in1 / out1 are NULL arrays where the path has no such buffer.
int srft_run_batched(const srft_plan_t* const* plans, const void* const* in0, const void* const* in1,
                     void* const* out0, void* const* out1, const int64_t* n_vec, int count, bool write_path,
                     hipStream_t st) {
    if (count < 0) return SRFT_ERR_BAD_N;
    if (count == 0) return SRFT_OK;
    if (!plans || !in0 || !out0 || !n_vec || (write_path ? !out1 : !in1)) return SRFT_ERR_NULL;
    bool lines = true;
    // validate everything before the first launch: a bad segment must not leave half a batch enqueued
    for (int i = 0; i < count; ++i) {
        if (!plans[i]) return SRFT_ERR_NULL;
        if (!srft_plans_compatible(plans[i], plans[0])) return SRFT_ERR_MISMATCH;
        if (n_vec[i] < 0 || n_vec[i] > kMaxVectors) return SRFT_ERR_BAD_N;
        if (n_vec[i] == 0) continue;
        const void* small = write_path ? (const void*)out1[i] : in1[i];       // the scales
        if (!in0[i] || !out0[i] || !small) return SRFT_ERR_NULL;
        if (!srft_aligned(in0[i], 16) || !srft_aligned(out0[i], 16) || !srft_aligned(small, 4)) return SRFT_ERR_ALIGN;
        lines &= srft_aligned(out0[i], 64);
    }
    srft_batch_even even;
    if (even_batch(plans, in0, out0, write_path ? (const void* const*)out1 : in1, n_vec, count, write_path, lines, &even)) {
        int threads = 0;
        const long long tiles = (even.n_vec + kTileVecs - 1) / kTileVecs * count;
        const batched_kernels_t kernel = batched_kernels(plans[0], write_path, tiles, lines, &threads);
        if (!kernel.even) return SRFT_ERR_BAD_D;
        return srft_launch(kernel.even, dim3((unsigned)srft_even_grid(even.shape, count)), threads, st, even, plans[0]->gw);
    }
    srft_batch_many a;
    int k = 0;
    for (int i = 0; i <= count; ++i) {
        if (i < count && n_vec[i] > 0) {
            srft_segment& s = a.seg[k++];
            s.frag = write_path ? srft_plan_write_table(plans[i]) : srft_plan_read_table(plans[i]);
            s.in = in0[i];
            s.out = out0[i];
            s.scales = (float*)(write_path ? out1[i] : in1[i]);
            s.n_vec = n_vec[i];
            s.unscale = write_path ? plans[i]->unscale_w : srft_plan_read_unscale(plans[i]);
        }
        if (k == kMaxBatch || (i == count && k > 0)) {
            const int rc = launch_batched(plans[0], a, k, write_path, lines, st);
            if (rc != SRFT_OK) return rc;
            k = 0;
        }
    }
    return SRFT_OK;
}

extern "C" {

int srft_kv_quantize(const srft_plan_t* plan, const void* x_f16_dev, int64_t n_vec, uint8_t* codes_dev,
                     float* scales_dev, void* hip_stream) {
    if (!plan) return SRFT_ERR_NULL;
    if (n_vec < 0 || n_vec > kMaxVectors) return SRFT_ERR_BAD_N;
    if (n_vec == 0) return SRFT_OK;
    if (!x_f16_dev || !codes_dev || !scales_dev) return SRFT_ERR_NULL;
    if (!srft_aligned(x_f16_dev, 16) || !srft_aligned(codes_dev, 16) || !srft_aligned(scales_dev, 4)) return SRFT_ERR_ALIGN;
    return launch_quantize(plan, x_f16_dev, n_vec, codes_dev, scales_dev, nullptr, kOutCodes, (hipStream_t)hip_stream);
}

int srft_kv_quantize_butterfly(const srft_plan_t* plan, const void* x_f16_dev, int64_t n_vec, uint8_t* codes_dev,
                               float* scales_dev, void* hip_stream) {
    if (!plan) return SRFT_ERR_NULL;
    if (plan->d != 128 && plan->d != 256) return SRFT_ERR_BAD_D;
    if (plan->gm != kGroup32) return SRFT_ERR_BAD_GROUP;
    if (plan->bits != 4) return SRFT_ERR_BAD_BITS;
    if (plan->transform != SRFT_TRANSFORM_DFT) return SRFT_ERR_BAD_TRANSFORM;
    if (n_vec < 0 || n_vec > kMaxVectors) return SRFT_ERR_BAD_N;
    if (n_vec == 0) return SRFT_OK;
    if (!x_f16_dev || !codes_dev || !scales_dev || !plan->bfly) return SRFT_ERR_NULL;
    if (!srft_aligned(x_f16_dev, 16) || !srft_aligned(codes_dev, 16) || !srft_aligned(scales_dev, 16)) return SRFT_ERR_ALIGN;
    return srft_launch_quantize_butterfly(plan->d, plan->bfly, x_f16_dev, n_vec, codes_dev, scales_dev, plan->max_wgs,
                                          (hipStream_t)hip_stream);
}

int srft_kv_forward_f32(const srft_plan_t* plan, const void* x_f16_dev, int64_t n_vec, float* w_f32_dev,
                        void* hip_stream) {
    if (!plan) return SRFT_ERR_NULL;
    if (n_vec < 0 || n_vec > kMaxVectors) return SRFT_ERR_BAD_N;
    if (n_vec == 0) return SRFT_OK;
    if (!x_f16_dev || !w_f32_dev) return SRFT_ERR_NULL;
    if (!srft_aligned(x_f16_dev, 16) || !srft_aligned(w_f32_dev, 16)) return SRFT_ERR_ALIGN;
    return launch_quantize(plan, x_f16_dev, n_vec, nullptr, nullptr, w_f32_dev, kOutRaw, (hipStream_t)hip_stream);
}

int srft_kv_channel_absmax(const srft_plan_t* plan, const void* x_f16_dev, int64_t n_vec, float* amax_dev,
                           void* hip_stream) {
    if (!plan) return SRFT_ERR_NULL;
    if (n_vec < 0 || n_vec > kMaxVectors) return SRFT_ERR_BAD_N;
    if (n_vec == 0) return SRFT_OK;
    if (!x_f16_dev || !amax_dev) return SRFT_ERR_NULL;
    if (!srft_aligned(x_f16_dev, 16) || !srft_aligned(amax_dev, 4)) return SRFT_ERR_ALIGN;
    return launch_quantize(plan, x_f16_dev, n_vec, nullptr, nullptr, amax_dev, kOutAmax, (hipStream_t)hip_stream);
}

int64_t srft_scores_workspace_bytes(const srft_plan_t* plan) {
    if (!plan) return SRFT_ERR_NULL;
    // (the kernel needs none; callers keep buffers of this size)
    return (int64_t)(plan->d / 16) * 2 * 64 * 16 + (int64_t)4096 * 64 * 4;
}

static int scores_check(const srft_plan_t* plan, const void* q_f16_dev, int n_q, const uint8_t* codes_dev,
                        const float* scales_dev, int64_t n_keys, const float* scores_dev) {
    if (!plan) return SRFT_ERR_NULL;
    if (plan->d % 64 != 0) return SRFT_ERR_BAD_D;
    if (plan->bits != 4) return SRFT_ERR_BAD_BITS;
    if (plan->gm == kGroup16) return SRFT_ERR_BAD_GROUP;
    if (n_q < 1 || n_q > 32 || n_keys < 0 || n_keys > kMaxVectors) return SRFT_ERR_BAD_N;
    if (n_keys == 0) return SRFT_OK;
    if (!q_f16_dev || !codes_dev || !scales_dev || !scores_dev) return SRFT_ERR_NULL;
    if (!srft_aligned(q_f16_dev, 16) || !srft_aligned(codes_dev, 16) || !srft_aligned(scales_dev, 4) || !srft_aligned(scores_dev, 4))
        return SRFT_ERR_ALIGN;
    return SRFT_OK;
}

int srft_kv_scores(const srft_plan_t* plan, const void* q_f16_dev, int n_q, const uint8_t* codes_dev,
                   const float* scales_dev, int64_t n_keys, float* scores_dev, void* workspace_dev, void* hip_stream) {
    const int rc = scores_check(plan, q_f16_dev, n_q, codes_dev, scales_dev, n_keys, scores_dev);
    if (n_keys == 0 && rc == SRFT_OK) return SRFT_OK;
    // (the workspace is not used; what was refused without a proper one still is)
    if ((rc == SRFT_OK || rc == SRFT_ERR_ALIGN) && !workspace_dev) return SRFT_ERR_NULL;
    if (rc == SRFT_OK && !srft_aligned(workspace_dev, 16)) return SRFT_ERR_ALIGN;
    if (rc != SRFT_OK) return rc;
    return srft_launch_scores(plan, q_f16_dev, n_q, codes_dev, scales_dev, n_keys, scores_dev, (hipStream_t)hip_stream);
}

int srft_kv_scores_static(const srft_plan_t* plan, const void* q_f16_dev, int n_q, const uint8_t* codes_dev,
                          const float* scales_dev, int64_t n_keys, float* scores_dev, void* hip_stream) {
    if (!plan) return SRFT_ERR_NULL;
    const int rc = scores_check(plan, q_f16_dev, n_q, codes_dev, scales_dev, n_keys, scores_dev);
    if (rc != SRFT_OK || n_keys == 0) return rc;
    return srft_launch_scores(plan, q_f16_dev, n_q, codes_dev, scales_dev, n_keys, scores_dev, (hipStream_t)hip_stream);
}

static int attend_supported(const srft_plan_t* plan) {
    if (plan->d % 64 != 0) return SRFT_ERR_BAD_D;
    if (plan->bits != 4) return SRFT_ERR_BAD_BITS;
    if (plan->gm == kGroup16) return SRFT_ERR_BAD_GROUP;
    return SRFT_OK;
}

int64_t srft_attend_workspace_bytes(const srft_plan_t* plan) {
    if (!plan) return SRFT_ERR_NULL;
    return (int64_t)srft_attend_workspace_floats(plan->d) * 4;
}

int srft_kv_attend(const srft_plan_t* plan, const float* weights_f32_dev, int n_q, const uint8_t* codes_dev,
                   const float* scales_dev, int64_t n_keys, float* out_f32_dev, void* workspace_dev, void* hip_stream) {
    if (!plan) return SRFT_ERR_NULL;
    const int rc = attend_supported(plan);
    if (rc != SRFT_OK) return rc;
    if (n_q < 1 || n_q > 32 || n_keys < 1 || n_keys > kMaxVectors) return SRFT_ERR_BAD_N;
    if (!weights_f32_dev || !codes_dev || !scales_dev || !out_f32_dev || !workspace_dev) return SRFT_ERR_NULL;
    if (!srft_aligned(weights_f32_dev, 4) || !srft_aligned(codes_dev, 16) || !srft_aligned(scales_dev, 4) ||
        !srft_aligned(out_f32_dev, 4) || !srft_aligned(workspace_dev, 16))
        return SRFT_ERR_ALIGN;
    return srft_launch_attend(plan, weights_f32_dev, n_q, codes_dev, scales_dev, n_keys, out_f32_dev,
                              (float*)workspace_dev, (hipStream_t)hip_stream);
}

int64_t srft_decode_attention_workspace_bytes(const srft_plan_t* plan_k, const srft_plan_t* plan_v, int n_q,
                                              int64_t n_keys) {
    if (!plan_k || !plan_v) return SRFT_ERR_NULL;
    if (n_q < 1 || n_q > 32 || n_keys < 1 || n_keys > kMaxVectors) return SRFT_ERR_BAD_N;
    // (More than the one-pass kernels use, which is checked against the last term where they are launched.  The size stays what
    // it was: programs take it as large as their longest context once and keep it for all their calls.)
    const int64_t scores = ((int64_t)n_q * n_keys * 4 + 255) / 256 * 256;
    return scores + 8192 + std::max(srft_scores_workspace_bytes(plan_k), srft_attend_workspace_bytes(plan_v));
}

int srft_kv_decode_attention(const srft_plan_t* plan_k, const srft_plan_t* plan_v, const void* q_f16_dev, int n_q,
                             const uint8_t* k_codes_dev, const float* k_scales_dev, const uint8_t* v_codes_dev,
                             const float* v_scales_dev, int64_t n_keys, float softmax_scale, float* out_f32_dev,
                             void* workspace_dev, void* hip_stream) {
    if (!plan_k || !plan_v) return SRFT_ERR_NULL;
    int rc = attend_supported(plan_v);
    if (rc != SRFT_OK) return rc;
    if (plan_k->d != plan_v->d || plan_k->device != plan_v->device) return SRFT_ERR_MISMATCH;
    if (n_q < 1 || n_q > 32 || n_keys < 1 || n_keys > kMaxVectors || !std::isfinite(softmax_scale)) return SRFT_ERR_BAD_N;
    if (!out_f32_dev || !workspace_dev || !v_codes_dev || !v_scales_dev) return SRFT_ERR_NULL;
    if (!srft_aligned(workspace_dev, 256) || !srft_aligned(out_f32_dev, 4) || !srft_aligned(v_codes_dev, 16) ||
        !srft_aligned(v_scales_dev, 4))
        return SRFT_ERR_ALIGN;
    if (plan_k->bits != 4) return SRFT_ERR_BAD_BITS;
    if (plan_k->gm == kGroup16) return SRFT_ERR_BAD_GROUP;
    if (!q_f16_dev || !k_codes_dev || !k_scales_dev) return SRFT_ERR_NULL;
    if (!srft_aligned(q_f16_dev, 16) || !srft_aligned(k_codes_dev, 16) || !srft_aligned(k_scales_dev, 4)) return SRFT_ERR_ALIGN;
    return srft_launch_decode_attention(plan_k, plan_v, q_f16_dev, n_q, k_codes_dev, k_scales_dev, v_codes_dev, v_scales_dev,
                                        n_keys, softmax_scale, out_f32_dev, workspace_dev, (hipStream_t)hip_stream);
}

int srft_lambda_from_absmax(const float* amax_host, int d, float* lambda_host) {
    if (!amax_host || !lambda_host) return SRFT_ERR_NULL;
    if (d < 1) return SRFT_ERR_BAD_D;
    float top = 0.0f;
    for (int k = 0; k < d; ++k) {
        if (!std::isfinite(amax_host[k]) || amax_host[k] < 0.0f) return SRFT_ERR_BAD_LAMBDA;
        top = std::fmax(top, amax_host[k]);
    }
    // lambda_k = 1 / amax_k; channels below 2^-16 of the largest are held there, which keeps max/min of lambda
    // within what srft_plan_create accepts; an all-zero batch gives all ones
    const float floor_ = std::ldexp(top, -16);
    for (int k = 0; k < d; ++k) lambda_host[k] = top > 0.0f ? 1.0f / std::fmax(amax_host[k], floor_) : 1.0f;
    return SRFT_OK;
}

int srft_kv_dequantize(const srft_plan_t* plan, const uint8_t* codes_dev, const float* scales_dev, int64_t n_vec,
                       void* out_f16_dev, void* hip_stream) {
    if (!plan) return SRFT_ERR_NULL;
    if (n_vec < 0 || n_vec > kMaxVectors) return SRFT_ERR_BAD_N;
    if (n_vec == 0) return SRFT_OK;
    if (!codes_dev || !scales_dev || !out_f16_dev) return SRFT_ERR_NULL;
    if (!srft_aligned(codes_dev, 16) || !srft_aligned(scales_dev, 4) || !srft_aligned(out_f16_dev, 16)) return SRFT_ERR_ALIGN;
    return launch_dequantize(plan, codes_dev, scales_dev, n_vec, out_f16_dev, (hipStream_t)hip_stream);
}

int srft_kv_quantize_batched(const srft_plan_t* const* plans, const void* const* x_f16_dev, const int64_t* n_vec,
                             uint8_t* const* codes_dev, float* const* scales_dev, int count, void* hip_stream) {
    return srft_run_batched(plans, x_f16_dev, nullptr, (void* const*)codes_dev, (void* const*)scales_dev, n_vec, count,
                       true, (hipStream_t)hip_stream);
}

int srft_kv_dequantize_batched(const srft_plan_t* const* plans, const uint8_t* const* codes_dev,
                               const float* const* scales_dev, const int64_t* n_vec, void* const* out_f16_dev,
                               int count, void* hip_stream) {
    return srft_run_batched(plans, (const void* const*)codes_dev, (const void* const*)scales_dev, out_f16_dev, nullptr,
                       n_vec, count, false, (hipStream_t)hip_stream);
}

const char* srft_status_string(int status) {
    switch (status) {
        case SRFT_OK: return "ok";
        case SRFT_ERR_NULL: return "required pointer is NULL";
        case SRFT_ERR_BAD_D: return "unsupported head dimension (need a multiple of 32 in [32, 256])";
        case SRFT_ERR_BAD_GROUP: return "unsupported group size (need 16, or a multiple of 32 that divides d)";
        case SRFT_ERR_BAD_LAMBDA: return "lambda must be finite, > 0 and span at most 2^16";
        case SRFT_ERR_ALIGN: return "device pointer is misaligned";
        case SRFT_ERR_HIP: return "HIP call failed (see srft_last_hip_error)";
        case SRFT_ERR_BAD_N: return "negative or malformed size";
        case SRFT_ERR_MISMATCH: return "plans of one call must share d, group size, code width and device";
        case SRFT_ERR_BAD_BITS: return "unsupported code width (need 4 or 8 bits)";
        case SRFT_ERR_BAD_TRANSFORM: return "unknown transform";
        default: return "unknown status";
    }
}

}  // extern "C"
