// cache.hip -- cache manager: host bookkeeping around the batched kernels and the flush (int4 store, fp16 residual window,
// dequantized view), and the small scatter kernel that places new tokens in the paged view.
#include <algorithm>
#include <memory>

#include "common.h"
#include "launch_shape.h"

namespace {

// Cache append: the new tokens of every plan, [n_seq][t_all][units] 16-byte units each, of which t go to their place in the
// paged fp16 view [block][n_seq][R][units]: token slot0 + j of sequence q lands in block block0 + (slot0 + j) / R, slot
// (slot0 + j) % R.  One thread per unit, blockIdx.y the plan, blockIdx.z the first sequence.  A decode step moves a few
// kilobytes, so the launch is all there is: 32-bit index arithmetic (one token of 2 sequences x 56 plans: 2.9 -> 2.3 us on the
// device) and no table of addresses where they lie a constant step apart (72 bytes of arguments against 1 KB: 3.0 against 4.2 us
// of the host; a prompt of 1000 tokens and 24 steps over 56 plans, with the conversions' launches, 151 -> 135 us; 85 to
// 97 with a flush of its own, see cache_flush.h).  A prompt is a
// copy at 4.7 TB/s.
struct scatter_args {
    const uint4* in[kMaxBatch];
    uint4* out[kMaxBatch];
    __device__ const uint4* from(int plan) const { return in[plan]; }
    __device__ uint4* to(int plan) const { return out[plan]; }
};
struct scatter_even {               // addresses a constant number of bytes apart
    const char* in;
    char* out;
    long long in_step, out_step;
    __device__ const uint4* from(int plan) const { return reinterpret_cast<const uint4*>(in + plan * in_step); }
    __device__ uint4* to(int plan) const { return reinterpret_cast<uint4*>(out + plan * out_step); }
};
template <class A>
__global__ void __launch_bounds__(256)
srft_cache_scatter_kernel(const A a, int n_seq, unsigned t, long long t_all, unsigned units, unsigned R,
                          long long block0, unsigned slot0) {
    const uint4* const in = a.from(blockIdx.y);
    uint4* const out = a.to(blockIdx.y);
    for (int seq = blockIdx.z; seq < n_seq; seq += gridDim.z)
        for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < t * units; i += gridDim.x * blockDim.x) {
            const unsigned tok = i / units, u = i % units, at = slot0 + tok, page = at / R, slot = at % R;
            out[(((block0 + page) * n_seq + seq) * R + slot) * units + u] = in[seq * t_all * units + i];
        }
}

}  // namespace

extern "C" {

int srft_cache_create(srft_cache_t** out, const srft_plan_t* const* plans, int n_plans, int n_seq,
                      int64_t capacity_tokens, int residual_tokens, uint8_t* const* codes_dev,
                      float* const* scales_dev, void* const* view_f16_dev) {
    if (!out) return SRFT_ERR_NULL;
    *out = nullptr;
    if (!plans || !codes_dev || !scales_dev || !view_f16_dev) return SRFT_ERR_NULL;
    if (n_plans < 1 || n_seq < 1 || residual_tokens < 1 || capacity_tokens < residual_tokens ||
        capacity_tokens % residual_tokens != 0 || capacity_tokens * n_seq > kMaxVectors)
        return SRFT_ERR_BAD_N;
    for (int i = 0; i < n_plans; ++i) {
        if (!plans[i] || !codes_dev[i] || !scales_dev[i] || !view_f16_dev[i]) return SRFT_ERR_NULL;
        if (!srft_plans_compatible(plans[i], plans[0])) return SRFT_ERR_MISMATCH;
        if (!srft_aligned(codes_dev[i], 16) || !srft_aligned(scales_dev[i], 4) || !srft_aligned(view_f16_dev[i], 16))
            return SRFT_ERR_ALIGN;
    }
    return srft_no_throw([&] {
        auto c = std::make_unique<srft_cache>();
        c->plans.assign(plans, plans + n_plans);
        c->codes.assign(codes_dev, codes_dev + n_plans);
        c->scales.assign(scales_dev, scales_dev + n_plans);
        c->view.assign(view_f16_dev, view_f16_dev + n_plans);
        c->n_seq = n_seq;
        c->R = residual_tokens;
        c->capacity = capacity_tokens;
        *out = c.release();
        return (int)SRFT_OK;
    });
}

int srft_cache_destroy(srft_cache_t* cache) {
    delete cache;
    return SRFT_OK;
}

int64_t srft_cache_tokens(const srft_cache_t* cache) { return cache ? cache->tokens : SRFT_ERR_NULL; }
int64_t srft_cache_quantized_tokens(const srft_cache_t* cache) { return cache ? cache->quantized : SRFT_ERR_NULL; }

// quantize (and read back into the view) or only read back the tokens [first, first + count) of every plan;
// both are multiples of R, so the range is contiguous in the paged layout
static int cache_convert(const srft_cache* c, int64_t first, int64_t count, bool quantize, hipStream_t st) {
    const size_t np = c->plans.size();
    const int d = c->plans[0]->d, G = d / c->plans[0]->g;
    const int64_t v0 = first * c->n_seq, nv = count * c->n_seq;          // vectors
    std::vector<const void*> x(np), cd(np), sc(np);
    std::vector<void*> xo(np), cdo(np), sco(np);
    std::vector<int64_t> n(np, nv);
    for (size_t i = 0; i < np; ++i) {
        xo[i] = (char*)c->view[i] + v0 * d * 2;
        cdo[i] = c->codes[i] + v0 * (d * c->plans[0]->bits / 8);
        sco[i] = c->scales[i] + v0 * G;
        x[i] = xo[i];
        cd[i] = cdo[i];
        sc[i] = sco[i];
    }
    if (quantize) {
        const int rc = srft_run_batched(c->plans.data(), x.data(), nullptr, cdo.data(), sco.data(), n.data(), (int)np,
                                   true, st);
        if (rc != SRFT_OK) return rc;
    }
    return srft_run_batched(c->plans.data(), cd.data(), sc.data(), xo.data(), nullptr, n.data(), (int)np, false, st);
}

// The append of t tokens that fills `count` tokens of pages per sequence, without a copy into the view in front (cache_flush.h):
// one launch, or two, the second one the read path's.  False: not for this cache, its buffers or its sizes.
static bool cache_flush(const srft_cache* c, const void* const* fresh, int t, int64_t count, hipStream_t st, int* rc) {
    const int np = (int)c->plans.size();
    const srft_plan* p = c->plans[0];
    const int64_t page_rows = (int64_t)c->n_seq * c->R, n_vec = count * c->n_seq, v0 = c->quantized * c->n_seq;
    if (!p->entry || !srft_flush_fits(n_vec, page_rows, c->n_seq, t, p->d / 8)) return false;
    srft_flush a;
    if (!srft_even_step(fresh, np, &a.fresh_step) || !srft_even_step(c->view.data(), np, &a.view_step) ||
        !srft_even_step((const void* const*)c->codes.data(), np, &a.codes_step) ||
        !srft_even_step((const void* const*)c->scales.data(), np, &a.scales_step))
        return false;
    a.plan_step = np > 1 ? (long long)((uintptr_t)c->plans[1]->entry - (uintptr_t)p->entry) : 0;
    for (int i = 1; i < np; ++i)
        if (!c->plans[i]->entry || (uintptr_t)c->plans[i]->entry - (uintptr_t)c->plans[i - 1]->entry != (uintptr_t)a.plan_step) return false;
    int threads = 0;
    const long long tiles = (n_vec + kTileVecs - 1) / kTileVecs;
    const bool staged = !p->fold_q && !p->fold4_q && srft_flush_staged(p->d, tiles * np);
    const flush_kernels_t kernels = srft_plan_flush_kernels(p, &threads, staged);
    const bool whole = kernels.whole && tiles * np <= (long long)srft_flush_whole_tiles(p->d, p->g) * p->grid_flush;
    const long long budget = p->max_wgs > 0 ? p->max_wgs : whole ? p->grid_flush : staged ? p->grid_staged : p->grid_q;
    if (np > budget) return false;
    const long long blocks = std::min(tiles, budget / np);
    if (blocks * np * blocks >= (1LL << 31)) return false;
    a.shape = srft_even_spread(tiles, np, budget, (int)blocks);
    a.plan = p->entry;
    a.fresh = (const char*)fresh[0];
    a.view = (char*)c->view[0] + v0 * p->d * 2;
    a.codes = (char*)c->codes[0] + v0 * (p->d * p->bits / 8);
    a.scales = (char*)(c->scales[0] + v0 * (p->d / p->g));
    a.n_vec = (int)n_vec;
    a.page_rows = (int)page_rows;
    a.R = c->R;
    a.held = (int)(c->tokens - c->quantized);
    a.t_all = t;
    a.tail = (int)(a.held + t - count);
    a.page_magic = srft_even_magic(a.page_rows);
    a.slot_magic = srft_even_magic(a.R);
    a.gw = p->gw;
    *rc = srft_launch(whole ? kernels.whole : kernels.write, dim3((unsigned)srft_even_grid(a.shape, np)), threads, st, a);
    if (*rc == SRFT_OK && !whole) *rc = srft_no_throw([&] { return cache_convert(c, c->quantized, count, false, st); });
    return true;
}

int srft_cache_append(srft_cache_t* cache, const void* const* new_f16_dev, int t, void* hip_stream) {
    if (!cache) return SRFT_ERR_NULL;
    if (t < 0 || cache->tokens + t > cache->capacity) return SRFT_ERR_BAD_N;
    if (t == 0) return SRFT_OK;
    if (!new_f16_dev) return SRFT_ERR_NULL;
    const size_t np = cache->plans.size();
    for (size_t i = 0; i < np; ++i) {
        if (!new_f16_dev[i]) return SRFT_ERR_NULL;
        if (!srft_aligned(new_f16_dev[i], 16)) return SRFT_ERR_ALIGN;
    }
    hipStream_t st = (hipStream_t)hip_stream;
    const int units = cache->plans[0]->d / 8;
    const int64_t full = (cache->tokens + t) / cache->R * cache->R;
    if (int rc; full > cache->quantized && cache_flush(cache, new_f16_dev, t, full - cache->quantized, st, &rc)) {
        if (rc != SRFT_OK) return rc;
        cache->tokens += t;
        cache->quantized = full;
        return SRFT_OK;
    }
    // 1. the new tokens join the window: an exact fp16 copy into the view
    scatter_even even;
    const bool is_even = np <= 4096 && srft_even_step(new_f16_dev, (int)np, &even.in_step) &&
                         srft_even_step(cache->view.data(), (int)np, &even.out_step);
    const size_t most = is_even ? np : kMaxBatch;
    for (int part = 0; part < srft_copy_launches(t); ++part)
        for (size_t p0 = 0; p0 < np; p0 += most) {
            const int64_t t0 = srft_copy_first(part);
            const unsigned n = srft_copy_tokens(part, t);
            const int plans = (int)std::min<size_t>(most, np - p0);
            const unsigned threads = std::min(256u, (n * units + 63) / 64 * 64);
            const int seqs = std::min(cache->n_seq, 64);     // (the grid: at most about 16 workgroups per compute unit)
            const unsigned blocks = std::max(1u, std::min((n * units + threads - 1) / threads, 4096u / (plans * seqs)));
            const int64_t pos = cache->tokens + t0;
            const auto copy = [&](auto kernel, const auto& a) {
                return srft_launch(kernel, dim3(blocks, plans, seqs), (int)threads, st, a, cache->n_seq, n, (long long)t,
                                   (unsigned)units, (unsigned)cache->R, (long long)(pos / cache->R), (unsigned)(pos % cache->R));
            };
            int rc;
            if (is_even) {
                even.in = (const char*)new_f16_dev[0] + (size_t)t0 * units * 16;
                even.out = (char*)cache->view[0];
                rc = copy(srft_cache_scatter_kernel<scatter_even>, even);
            } else {
                scatter_args a;
                for (int k = 0; k < plans; ++k) {
                    a.in[k] = (const uint4*)new_f16_dev[p0 + k] + (size_t)t0 * units;
                    a.out[k] = (uint4*)cache->view[p0 + k];
                }
                rc = copy(srft_cache_scatter_kernel<scatter_args>, a);
            }
            if (rc != SRFT_OK) return rc;
        }
    cache->tokens += t;
    // 2. (where cache_flush does not apply) every window that is now full is quantized into the store and replaced, in the view, by
    //    what the store decodes to (the window is "re-quantized when full"; the dequantized prefix is refreshed only here)
    if (full > cache->quantized) {
        const int rc = srft_no_throw([&] { return cache_convert(cache, cache->quantized, full - cache->quantized, true, st); });
        if (rc != SRFT_OK) return rc;
        cache->quantized = full;
    }
    return SRFT_OK;
}

int srft_cache_rebuild_view(srft_cache_t* cache, void* hip_stream) {
    if (!cache) return SRFT_ERR_NULL;
    if (cache->quantized == 0) return SRFT_OK;
    return srft_no_throw([&] { return cache_convert(cache, 0, cache->quantized, false, (hipStream_t)hip_stream); });
}

}  // extern "C"
