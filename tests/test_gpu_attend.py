"""GPU parity of the value side of attention over the stored cache (srft_kv_attend, srft_kv_decode_attention) against
the oracle's plain definitions."""
import numpy as np
import pytest
import torch

from oracle import srft_oracle as O
from paper_2605_05699_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2605_05699_amd import binding
    binding.lib()
    return binding


def _attend(B, plan, w, codes, scales):
    out = torch.full((w.shape[0], plan.d), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(B.lib().srft_attend_workspace_bytes(plan.handle), dtype=torch.uint8, device="cuda")
    B.srft_kv_attend(plan.handle, w, codes, scales, out, ws)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def _tolerance(w64, vals64):
    # the products w * scale are carried as fp16 hi + lo (2^-21 relative each), the sums are fp32 over at most a few
    # hundred tiles per workgroup and a few hundred workgroups, the inverse transform is fp32 over d terms: a few
    # 1e-6 of sum_t |w_t| max|v| covers all of it; the oracle is fp64
    return 6e-6 * np.abs(w64).sum(axis=1)[:, None] * np.abs(vals64).max() + 1e-30


@pytest.mark.parametrize("d", [64, 128, 192, 256])
@pytest.mark.parametrize("n_q,n_keys", [(1, 1), (8, 33), (32, 1000), (5, 4097), (3, 64), (12, 300), (16, 129), (17, 100)])
def test_attend_matches_the_definition(B, d, n_q, n_keys):
    g = 32
    vals = W.gaussian_with_outliers(n_keys, d, seed=3 * d + n_keys, outliers=1, gain=10.0)
    lam = W.lognormal_lambda(d, seed=d + 5)
    plan = B.Plan(d, g, 700 + d, lam)
    codes, scales = plan.quantize(torch.from_numpy(vals).cuda())
    rng = np.random.RandomState(n_q + n_keys)
    w = rng.rand(n_q, n_keys).astype(np.float32)
    w[0] = 0.0
    w[0, n_keys // 2] = 1.0                       # a one-hot row: that value's reconstruction
    if n_q > 1:
        w[1] = rng.standard_normal(n_keys).astype(np.float32)      # weights need not be probabilities
    got = _attend(B, plan, torch.from_numpy(w).cuda(), codes, scales)
    c, sc = codes.cpu().numpy(), scales.cpu().numpy()
    ref = O.attention_output(w, c, sc, plan.signs, lam, g)
    back = O.dequantize_f64(c, sc, plan.signs, lam, g)
    assert got.shape == (n_q, d) and np.isfinite(got).all()
    tol = _tolerance(w.astype(np.float64), back)
    assert np.all(np.abs(got - ref) <= tol), float((np.abs(got - ref) / tol).max())
    assert np.all(np.abs(got[0] - back[n_keys // 2]) <= tol[0])
    plan.close()


def test_attend_over_many_tiles_wide_groups_a_grid_cap_and_argument_checks(B):
    d, n_keys, n_q = 128, 200_003, 8
    vals = W.gaussian_with_outliers(n_keys, d, seed=4, outliers=1, gain=20.0)
    rng = np.random.RandomState(1)
    logits = rng.standard_normal((n_q, n_keys)) * 3.0
    w = O.softmax_rows(logits).astype(np.float32)
    wd = torch.from_numpy(w).cuda()
    for g in (32, 64, 128):
        lam = W.lognormal_lambda(d, seed=g)
        plan = B.Plan(d, g, 11, lam)
        codes, scales = plan.quantize(torch.from_numpy(vals).cuda())
        got = _attend(B, plan, wd, codes, scales)
        c, sc = codes.cpu().numpy(), scales.cpu().numpy()
        ref = O.attention_output(w, c, sc, plan.signs, lam, g)
        tol = _tolerance(w.astype(np.float64), O.dequantize_f64(c[:4096], sc[:4096], plan.signs, lam, g) * 1.5)
        assert np.all(np.abs(got - ref) <= tol), (g, float((np.abs(got - ref) / tol).max()))
        if g == 32:
            # fewer workgroups: another split of the keys, the same sums to rounding
            B.srft_plan_set_max_workgroups(plan.handle, 3)
            again = _attend(B, plan, wd, codes, scales)
            assert np.all(np.abs(again - ref) <= tol)
            B.srft_plan_set_max_workgroups(plan.handle, 0)
            twice = _attend(B, plan, wd, codes, scales)
            assert np.array_equal(twice, got)                     # fixed summation order: bitwise repeatable
            L = B.lib()
            ws = torch.empty(L.srft_attend_workspace_bytes(plan.handle), dtype=torch.uint8, device="cuda")
            out = torch.empty(n_q, d, dtype=torch.float32, device="cuda")
            args = (wd.data_ptr(), n_q, codes.data_ptr(), scales.data_ptr(), n_keys, out.data_ptr(), ws.data_ptr(), None)
            assert L.srft_kv_attend(None, *args) == -1
            assert L.srft_kv_attend(plan.handle, wd.data_ptr(), 33, *args[2:]) == -7
            assert L.srft_kv_attend(plan.handle, wd.data_ptr(), n_q, codes.data_ptr(), scales.data_ptr(), 0, out.data_ptr(), ws.data_ptr(), None) == -7
            assert L.srft_kv_attend(plan.handle, None, *args[1:]) == -1
            assert L.srft_kv_attend(plan.handle, wd.data_ptr(), n_q, codes.data_ptr() + 1, *args[3:]) == -5
        plan.close()
    p96 = B.Plan(96, 32, 1)
    assert B.lib().srft_attend_workspace_bytes(p96.handle) > 0
    assert B.lib().srft_kv_attend(p96.handle, wd.data_ptr(), 1, wd.data_ptr(), wd.data_ptr(), 1, wd.data_ptr(), wd.data_ptr(), None) == -2
    p96.close()


@pytest.mark.parametrize("d,n_q,n_keys", [(128, 8, 5000), (256, 4, 1234), (64, 32, 777), (128, 16, 70001), (192, 9, 40)])
def test_decode_attention_matches_the_definition(B, d, n_q, n_keys):
    g = 32
    k = W.gaussian_with_outliers(n_keys, d, seed=d + 1, outliers=1, gain=15.0)
    v = W.gaussian_with_outliers(n_keys, d, seed=d + 2, outliers=0)
    q = W.gaussian_with_outliers(n_q, d, seed=d + 3, outliers=1, gain=4.0)
    lam_k, lam_v = W.lognormal_lambda(d, seed=1), W.lognormal_lambda(d, seed=2)
    pk, pv = B.Plan(d, g, 21, lam_k), B.Plan(d, g, 22, lam_v)
    kc, ks = pk.quantize(torch.from_numpy(k).cuda())
    vc, vs = pv.quantize(torch.from_numpy(v).cuda())
    scale = d ** -0.5
    out = torch.full((n_q, d), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(B.lib().srft_decode_attention_workspace_bytes(pk.handle, pv.handle, n_q, n_keys), dtype=torch.uint8,
                     device="cuda")
    B.srft_kv_decode_attention(pk.handle, pv.handle, torch.from_numpy(q).cuda(), kc, ks, vc, vs, scale, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    ref = O.decode_attention(q, kc.cpu().numpy(), ks.cpu().numpy(), pk.signs, lam_k, vc.cpu().numpy(), vs.cpu().numpy(),
                             pv.signs, lam_v, g, scale)
    vb = O.dequantize_f64(vc.cpu().numpy(), vs.cpu().numpy(), pv.signs, lam_v, g)
    # the scores carry an absolute error of about 4e-6 |q| |k| (test_gpu_scores.py); times softmax_scale it moves every
    # probability by that relative amount, and the output by at most twice that times max |v|; plus the weighted sum's own
    kb = O.dequantize_f64(kc.cpu().numpy(), ks.cpu().numpy(), pk.signs, lam_k, g)
    ds = 4e-6 * scale * np.linalg.norm(q.astype(np.float64), axis=1).max() * np.linalg.norm(kb, axis=1).max() + 2e-7
    tol = (2 * ds + 6e-6) * np.abs(vb).max() + 1e-30
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= tol, float(np.abs(got - ref).max() / tol)
    pk.close()
    pv.close()


def test_decode_attention_replayed_from_a_hip_graph_equals_the_eager_calls(B):
    """The entry point only enqueues kernels on the caller's stream (no allocation, no memset), so a caller may record
    it into a HIP graph.  Three replays, each after new queries were written into the captured buffer by ordinary eager
    work, must equal the eager call on the same inputs bit for bit (the summation order is fixed)."""
    d, g, n_q, n_keys = 128, 32, 8, 20_000
    k = W.gaussian_with_outliers(n_keys, d, seed=31, outliers=1, gain=15.0)
    v = W.gaussian_with_outliers(n_keys, d, seed=32, outliers=0)
    pk, pv = B.Plan(d, g, 41, W.lognormal_lambda(d, seed=3)), B.Plan(d, g, 42, W.lognormal_lambda(d, seed=4))
    kc, ks = pk.quantize(torch.from_numpy(k).cuda())
    vc, vs = pv.quantize(torch.from_numpy(v).cuda())
    scale = d ** -0.5
    q = torch.zeros(n_q, d, dtype=torch.float16, device="cuda")
    out = torch.zeros(n_q, d, dtype=torch.float32, device="cuda")
    nbytes = B.lib().srft_decode_attention_workspace_bytes(pk.handle, pv.handle, n_q, n_keys)
    ws, ws_eager = (torch.empty(nbytes, dtype=torch.uint8, device="cuda") for _ in range(2))
    q.copy_(torch.from_numpy(W.gaussian_with_outliers(n_q, d, seed=50, outliers=0)))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):              # one eager call on the capture stream first
        B.srft_kv_decode_attention(pk.handle, pv.handle, q, kc, ks, vc, vs, scale, out, ws, side)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        B.srft_kv_decode_attention(pk.handle, pv.handle, q, kc, ks, vc, vs, scale, out, ws, torch.cuda.current_stream())
    for rep in range(3):
        q.copy_(torch.from_numpy(W.gaussian_with_outliers(n_q, d, seed=60 + rep, outliers=1, gain=3.0)))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        eager = torch.empty_like(out)
        B.srft_kv_decode_attention(pk.handle, pv.handle, q, kc, ks, vc, vs, scale, eager, ws_eager)
        torch.cuda.synchronize()
        assert torch.equal(got, eager), rep
        assert torch.isfinite(got).all() and got.abs().max() > 0
    pk.close()
    pv.close()


@pytest.mark.parametrize("d,g,n_q,n_keys,cap,scale", [
    (128, 32, 1, 1, 0, 0.1), (128, 32, 16, 31, 0, 0.1), (64, 32, 17, 33, 0, 0.1),          # less than one tile, one key more
    (256, 32, 32, 768, 3, 0.1), (256, 32, 5, 769, 3, 0.1),                                 # last of the 32-key tiles, first of 64
    (192, 32, 16, 1537, 3, 0.1), (128, 64, 9, 3 * 512 + 65, 3, 0.1), (64, 64, 8, 5000, 1, 0.1),     # second and later tiles of a wavefront
    (256, 256, 4, 1000, 0, 0.1), (192, 96, 3, 200, 2, 0.1),                                # wide groups
    (128, 32, 8, 2000, 0, -0.1), (128, 32, 8, 300, 0, 0.0), (128, 32, 3, 16500, 300, 0.1),  # sign of the scale; more than 256 workgroups
])
def test_decode_attention_at_the_edges_of_its_tiles_and_grid(B, d, g, n_q, n_keys, cap, scale):
    k = W.gaussian_with_outliers(n_keys, d, seed=d + n_keys, outliers=1, gain=15.0)
    v = W.gaussian_with_outliers(n_keys, d, seed=d + n_keys + 1, outliers=0)
    q = W.gaussian_with_outliers(n_q, d, seed=d + n_keys + 2, outliers=1, gain=4.0)
    k[n_keys // 2] *= 8.0                              # a key that outweighs what came before it
    lam_k, lam_v = W.lognormal_lambda(d, seed=1), W.lognormal_lambda(d, seed=2)
    pk, pv = B.Plan(d, g, 23, lam_k), B.Plan(d, g, 24, lam_v)
    kc, ks = pk.quantize(torch.from_numpy(k).cuda())
    vc, vs = pv.quantize(torch.from_numpy(v).cuda())
    B.srft_plan_set_max_workgroups(pv.handle, cap)
    ws = torch.empty(B.lib().srft_decode_attention_workspace_bytes(pk.handle, pv.handle, n_q, n_keys), dtype=torch.uint8,
                     device="cuda")
    ws.fill_(0xFF)                                     # (NaN as floats: nothing is read that was not written)
    out = torch.full((n_q, d), float("nan"), dtype=torch.float32, device="cuda")
    B.srft_kv_decode_attention(pk.handle, pv.handle, torch.from_numpy(q).cuda(), kc, ks, vc, vs, scale, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    kc, ks, vc, vs = (t.cpu().numpy() for t in (kc, ks, vc, vs))
    ref = O.decode_attention(q, kc, ks, pk.signs, lam_k, vc, vs, pv.signs, lam_v, g, scale)
    kb, vb = O.dequantize_f64(kc, ks, pk.signs, lam_k, g), O.dequantize_f64(vc, vs, pv.signs, lam_v, g)
    # the bound of test_decode_attention_matches_the_definition
    ds = 4e-6 * abs(scale) * np.linalg.norm(q.astype(np.float64), axis=1).max() * np.linalg.norm(kb, axis=1).max() + 2e-7
    tol = (2 * ds + 6e-6) * np.abs(vb).max() + 1e-30
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= tol, float(np.abs(got - ref).max() / tol)
    pk.close()
    pv.close()


def test_decode_attention_keeps_weights_far_below_the_largest(B):
    """One key outweighs each of the others by about e^17, and there are enough of them that together they still matter:
    a weight below the smallest fp16 number (relative to the row's maximum) must not vanish."""
    d, g, n_keys = 64, 32, 200_000
    rng = np.random.RandomState(3)
    k = (0.02 * rng.standard_normal((n_keys, d))).astype(np.float16)
    q = np.ones((1, d), dtype=np.float16)
    k[12345] = np.float16(17.0 / 64 / 0.125)          # softmax_scale q.k = 17 for this key, about 0 for the others
    v = (1.0 + 0.1 * rng.standard_normal((n_keys, d))).astype(np.float16)
    v[12345] = 0.0                                    # so the output is what the others carry: about n e^-17 / (1 + n e^-17)
    pk, pv = B.Plan(d, g, 31), B.Plan(d, g, 32)
    kc, ks = pk.quantize(torch.from_numpy(k).cuda())
    vc, vs = pv.quantize(torch.from_numpy(v).cuda())
    out = torch.empty(1, d, dtype=torch.float32, device="cuda")
    ws = torch.empty(B.lib().srft_decode_attention_workspace_bytes(pk.handle, pv.handle, 1, n_keys), dtype=torch.uint8, device="cuda")
    B.srft_kv_decode_attention(pk.handle, pv.handle, torch.from_numpy(q).cuda(), kc, ks, vc, vs, 0.125, out, ws)
    torch.cuda.synchronize()
    ones = np.ones(d, dtype=np.float32)
    ref = O.decode_attention(q, kc.cpu().numpy(), ks.cpu().numpy(), pk.signs, ones, vc.cpu().numpy(), vs.cpu().numpy(),
                             pv.signs, ones, g, 0.125)
    # scores of size 17 in fp32 (2e-6 absolute), weights and sums as in the other tests
    assert np.abs(out.cpu().numpy() - ref).max() <= 3e-5 * np.abs(ref).max(), (np.abs(out.cpu().numpy() - ref).max(), np.abs(ref).max())
    assert 0.003 < np.abs(ref).max() < 0.1
    pk.close()
    pv.close()


def _decode_attention(B, pk, pv, q, kc, ks, vc, vs, scale):
    ws = torch.full((B.lib().srft_decode_attention_workspace_bytes(pk.handle, pv.handle, q.shape[0], kc.shape[0]),), 0xFF,
                    dtype=torch.uint8, device="cuda")                # (NaN as floats: nothing is read that was not written)
    out = torch.full((q.shape[0], pk.d), float("nan"), dtype=torch.float32, device="cuda")
    B.srft_kv_decode_attention(pk.handle, pv.handle, q, kc, ks, vc, vs, scale, out, ws)
    torch.cuda.synchronize()
    return out


# where the large scales are (keys of no weight), the power of two of the others
SPANS = {"before": (lambda t, n: t < n // 4, 0), "beside": (lambda t, n: t % 2 == 1, 0), "after": (lambda t, n: t >= n - n // 4, 0),
         "none, tiny scales": (lambda t, n: t < 0, -80), "none, large scales": (lambda t, n: t < 0, 40)}


@pytest.mark.parametrize("where", SPANS)
@pytest.mark.parametrize("d,n_q,n_keys,cap", [(64, 3, 4096, 1), (128, 8, 4096, 2), (256, 4, 4096, 2), (128, 5, 500, 2), (192, 17, 2048, 1)])
def test_decode_attention_of_values_whose_scales_span_many_powers(B, d, n_q, n_keys, cap, where):
    """Keys of no weight (e^-40 and less) with values 2^28 times the others', before, beside and after those that weigh: what
    the others carry must keep its 20 bits.  Tiles of 64 and of 32 keys, several tiles per wavefront."""
    rng = np.random.RandomState(d + n_keys)
    direction = rng.standard_normal(d)
    q = (np.outer(1.0 + 0.1 * np.arange(n_q), direction)).astype(np.float16)
    large, power = SPANS[where]
    loud = torch.from_numpy(large(np.arange(n_keys), n_keys)).cuda()
    # all keys that weigh are the same key: their scores are equal to the last bit, 40 above those of the others
    k = torch.from_numpy(np.tile(direction * 40.0 / (direction @ direction) / 0.125, (n_keys, 1)).astype(np.float16)).cuda()
    v = torch.from_numpy(W.gaussian_with_outliers(n_keys, d, seed=d, outliers=0)).cuda()
    pk, pv = B.Plan(d, 32, 41), B.Plan(d, 32, 42)
    kc, ks = pk.quantize(k)
    vc, vs = pv.quantize(v)
    ks[loud] = 0.0
    vs *= 2.0 ** power
    vs[loud] *= 2.0 ** 28
    B.srft_plan_set_max_workgroups(pv.handle, cap)
    got = _decode_attention(B, pk, pv, torch.from_numpy(q).cuda(), kc, ks, vc, vs, 0.125).double().cpu().numpy()
    ones = np.ones(d, dtype=np.float32)
    kc, ks, vc, vs = (t.cpu().numpy() for t in (kc, ks, vc, vs))
    weights = O.softmax_rows(O.attention_scores(q, kc, ks, pk.signs, ones, 32), 0.125)
    vb = O.dequantize_f64(vc, vs, pv.signs, ones, 32)
    tol = 6e-6 * (weights @ np.abs(vb)).max(axis=1, keepdims=True)       # of the weighted sums, see _tolerance
    err = np.abs(got - weights @ vb)
    assert np.all(err <= tol), float((err / tol).max())
    pk.close()
    pv.close()


# shapes at the edges of the decode attention's tiles (32 and 64 keys), of a wavefront's share and of its grid: d, g, n_q, n_keys, cap
EDGES = [(128, 32, 1, 1, 0), (128, 32, 16, 31, 0), (64, 32, 17, 33, 0), (256, 32, 32, 768, 3), (256, 32, 5, 769, 3), (192, 32, 16, 1537, 3),
         (128, 64, 9, 1601, 3), (64, 64, 8, 5000, 1), (256, 256, 4, 1000, 0), (192, 96, 3, 200, 2), (128, 32, 3, 16500, 300)]


def _plans_and_record(B, d, g, k, v, cap):
    lam_k, lam_v = W.lognormal_lambda(d, seed=1), W.lognormal_lambda(d, seed=2)
    pk, pv = B.Plan(d, g, 51, lam_k), B.Plan(d, g, 52, lam_v)
    record = (*pk.quantize(torch.from_numpy(k).cuda()), *pv.quantize(torch.from_numpy(v).cuda()))
    B.srft_plan_set_max_workgroups(pv.handle, cap)
    host = [t.cpu().numpy() for t in record]
    return pk, pv, record, O.dequantize_f64(*host[:2], pk.signs, lam_k, g), O.dequantize_f64(*host[2:], pv.signs, lam_v, g)


@pytest.mark.parametrize("d,g,n_q,n_keys,cap", EDGES)
def test_decode_attention_with_equal_weights_counts_every_key_once(B, d, g, n_q, n_keys, cap):
    """softmax_scale 0: the mean of the values, to the error of the weighted sum alone.  The last key and the first of the
    last tile are 100 times the others: one that is lost, or taken twice, shows at any length."""
    k = W.gaussian_with_outliers(n_keys, d, seed=d + n_keys, outliers=1, gain=15.0)
    v = W.gaussian_with_outliers(n_keys, d, seed=d + n_keys + 1, outliers=0)
    for t in {n_keys - 1, (n_keys - 1) // 32 * 32, (n_keys - 1) // 64 * 64}:
        v[t] *= 100.0
    q = W.gaussian_with_outliers(n_q, d, seed=d + n_keys + 2, outliers=1, gain=4.0)
    pk, pv, record, _, vb = _plans_and_record(B, d, g, k, v, cap)
    got = _decode_attention(B, pk, pv, torch.from_numpy(q).cuda(), *record, 0.0).double().cpu().numpy()
    tol = 6e-6 * np.abs(vb).mean(axis=0).max()               # of the weighted sums, see _tolerance
    assert np.abs(got - vb.mean(axis=0)).max() <= tol, float(np.abs(got - vb.mean(axis=0)).max() / tol)
    assert tol < 0.01 * np.abs(vb[-1]).max() / n_keys        # one key of the large ones is far above it
    pk.close()
    pv.close()


@pytest.mark.parametrize("d,g,n_q,n_keys,cap", [e for e in EDGES if e[3] > 500])
def test_decode_attention_where_the_maximum_keeps_growing(B, d, g, n_q, n_keys, cap):
    """Scores that rise by 1/2 from one stretch of keys to the next (and fall, in the second half of the queries), magnitudes of
    the values that go up and down by 2^10: every tile brings a new maximum, and what was summed before still counts."""
    direction = np.random.RandomState(d).standard_normal(d)
    level = 8.0 * np.arange(n_keys) // n_keys                # 0 .. 7
    k = (np.outer(0.5 * level, direction) / (direction @ direction)).astype(np.float16)
    v = (W.gaussian_with_outliers(n_keys, d, seed=d + n_keys, outliers=0).astype(np.float32) * 2.0 ** (5 * (level % 3))[:, None]).astype(np.float16)
    q = np.outer(np.where(2 * np.arange(n_q) >= n_q, -1.0, 1.0), direction).astype(np.float16)
    pk, pv, record, kb, vb = _plans_and_record(B, d, g, k, v, cap)
    got = _decode_attention(B, pk, pv, torch.from_numpy(q).cuda(), *record, 1.0).double().cpu().numpy()
    scores = q.astype(np.float64) @ kb.T
    weights = O.softmax_rows(scores, 1.0)
    # scores of up to 4 are off by 4e-6 |q| |k| (test_gpu_scores.py), per row; the weighted sums as in _tolerance
    ds = 4e-6 * np.linalg.norm(q.astype(np.float64), axis=1) * np.linalg.norm(kb, axis=1).max()
    tol = (2 * ds + 6e-6)[:, None] * (weights @ np.abs(vb)).max(axis=1, keepdims=True)
    err = np.abs(got - weights @ vb)
    assert np.all(err <= tol), float((err / tol).max())
    pk.close()
    pv.close()


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_what_is_not_finite_stays_with_its_query_or_its_key(B, bad):
    d, n_q, n_keys = 128, 20, 700
    k, v = (W.gaussian_with_outliers(n_keys, d, seed=s, outliers=0) for s in (1, 2))
    q = torch.from_numpy(W.gaussian_with_outliers(n_q, d, seed=3, outliers=0)).cuda()
    pk, pv, (kc, ks, vc, vs), _, _ = _plans_and_record(B, d, 32, k, v, 0)
    ws = torch.empty(B.lib().srft_scores_workspace_bytes(pk.handle), dtype=torch.uint8, device="cuda")

    def both(q, ks, vs):
        scores = torch.empty(n_q, n_keys, device="cuda")
        B.srft_kv_scores(pk.handle, q, kc, ks, scores, ws)
        return scores, _decode_attention(B, pk, pv, q, kc, ks, vc, vs, 0.09)

    scores, out = both(q, ks, vs)
    assert bool(torch.isfinite(scores).all()) and bool(torch.isfinite(out).all())
    qb, ksb, vsb = q.clone(), ks.clone(), vs.clone()
    qb[17, 5] = bad
    ksb[300, 2] = bad
    vsb[600, 1] = bad
    rest = torch.arange(n_q, device="cuda") != 17
    for got, good in zip(both(qb, ks, vs), (scores, out)):   # a query: its row and no other
        assert torch.equal(got[rest], good[rest]) and not bool(torch.isfinite(got[17]).any())
    got, attended = both(q, ksb, vs)                         # a key's scale: its score, and every softmax over it
    others = torch.arange(n_keys, device="cuda") != 300
    assert torch.equal(got[:, others], scores[:, others]) and not bool(torch.isfinite(got[:, 300]).any())
    assert not bool(torch.isfinite(attended[got[:, 300] != -bad]).any())
    assert not bool(torch.isfinite(both(q, ks, vsb)[1]).any())           # a value's scale: every sum over it
    pk.close()
    pv.close()


@pytest.mark.parametrize("n_q,cap", [(16, 6), (17, 6), (32, 7), (32, 1)])
def test_decode_attention_keeps_to_the_cap_on_workgroups(B, n_q, cap):
    """The scan leaves a maximum per query and workgroup, 1024 floats apart per query, at the start of the workspace; every
    16 queries have workgroups of their own."""
    d, n_keys = 128, 6000
    k, v, q = (W.gaussian_with_outliers(n, d, seed=n + s, outliers=0) for n, s in ((n_keys, 1), (n_keys, 2), (n_q, 3)))
    pk, pv, (kc, ks, vc, vs), kb, vb = _plans_and_record(B, d, 32, k, v, cap)
    ws = torch.full((B.lib().srft_decode_attention_workspace_bytes(pk.handle, pv.handle, n_q, n_keys),), 0xFF, dtype=torch.uint8, device="cuda")
    out = torch.empty(n_q, d, device="cuda")
    B.srft_kv_decode_attention(pk.handle, pv.handle, torch.from_numpy(q).cuda(), kc, ks, vc, vs, 0.09, out, ws)
    torch.cuda.synchronize()
    written = ~torch.isnan(ws[:32 * 1024 * 4].view(torch.float32).view(32, 1024))
    workgroups = sum(int(written[i].sum()) for i in range(0, n_q, 16))
    assert 1 <= workgroups <= max(cap, (n_q + 15) // 16)
    ref = O.softmax_rows(q.astype(np.float64) @ kb.T, 0.09) @ vb
    assert np.abs(out.cpu().numpy() - ref).max() <= 1e-4 * np.abs(vb).max()
    pk.close()
    pv.close()


@pytest.mark.parametrize("d", [64, 128, 192, 256])
@pytest.mark.parametrize("cap,n_keys", [(1, 32), (8, 256), (8, 264), (64, 4000), (65, 4000), (128, 5000), (129, 5000), (256, 20000),
                                        (257, 20000), (700, 50005)])
def test_decode_attention_whatever_the_number_of_workgroups_to_add(B, d, cap, n_keys):
    """One wavefront of a workgroup with keys, some, all of them; up to 256 workgroups to add and more: as one workgroup has it."""
    n_q = 5
    pk, pv = B.Plan(d, 32, 1, W.lognormal_lambda(d, seed=1)), B.Plan(d, 32, 2, W.lognormal_lambda(d, seed=2))
    gen = torch.Generator(device="cuda").manual_seed(d + cap)
    q = torch.randn(n_q, d, generator=gen, device="cuda").half()
    k, v = (p.quantize(torch.randn(n_keys, d, generator=gen, device="cuda").half()) for p in (pk, pv))
    ws = torch.empty(B.lib().srft_decode_attention_workspace_bytes(pk.handle, pv.handle, n_q, n_keys), dtype=torch.uint8, device="cuda")
    out = []
    for c in (1, cap):
        B.srft_plan_set_max_workgroups(pk.handle, c)
        o = torch.full((n_q, d), float("nan"), device="cuda")
        B.srft_kv_decode_attention(pk.handle, pv.handle, q, *k, *v, d ** -0.5, o, ws)
        out.append(o.double())
    # both sum the same fp32 products in other orders
    assert (out[0] - out[1]).abs().max() <= 4e-6 * out[0].abs().max()
    pk.close()
    pv.close()


@pytest.mark.parametrize("transforms", [("hadamard", "hadamard"), ("hadamard", "dft"), ("dft", "hadamard")])
@pytest.mark.parametrize("d,g,n_q,n_keys,cap,scale", [(64, 32, 5, 33, 0, 0.1), (64, 64, 17, 5000, 1, -0.1), (128, 32, 8, 1601, 0, 0.1),
                                                      (128, 128, 32, 900, 2, -0.1), (256, 32, 16, 769, 3, -0.1), (256, 32, 20, 4096, 0, 0.1)])
def test_decode_attention_of_hadamard_plans(B, transforms, d, g, n_q, n_keys, cap, scale):
    """Keys and values under either transform, both signs of the scale, one and two blocks of 16 queries."""
    k = W.gaussian_with_outliers(n_keys, d, seed=d + n_keys, outliers=1, gain=15.0)
    v = W.gaussian_with_outliers(n_keys, d, seed=d + n_keys + 1, outliers=0)
    q = W.gaussian_with_outliers(n_q, d, seed=d + n_keys + 2, outliers=1, gain=4.0)
    lam = [W.lognormal_lambda(d, seed=s) for s in (1, 2)]
    plans = [B.Plan(d, g, 61 + i, lam[i], transform=t) for i, t in enumerate(transforms)]
    record = [t for p, x in zip(plans, (k, v)) for t in p.quantize(torch.from_numpy(x).cuda())]
    B.srft_plan_set_max_workgroups(plans[1].handle, cap)
    got = _decode_attention(B, *plans, torch.from_numpy(q).cuda(), *record, scale).double().cpu().numpy()
    host = [t.cpu().numpy() for t in record]
    kb, vb = (O.dequantize_f64(*host[2 * i:2 * i + 2], plans[i].signs, lam[i], g, form="hadamard" if t == "hadamard" else "dense")
              for i, t in enumerate(transforms))
    ref = O.softmax_rows(q.astype(np.float64) @ kb.T, scale) @ vb
    # the bound of test_decode_attention_matches_the_definition
    ds = 4e-6 * abs(scale) * np.linalg.norm(q.astype(np.float64), axis=1).max() * np.linalg.norm(kb, axis=1).max() + 2e-7
    tol = (2 * ds + 6e-6) * np.abs(vb).max()
    assert np.abs(got - ref).max() <= tol, float(np.abs(got - ref).max() / tol)
    for p in plans:
        p.close()


# Tiles of 32 keys, by wavefronts in teams of d / 64 (up to 8 / team tiles a workgroup), of two (d = 256, up to 4) and alone: the
# last size of each form and the first of the next, at 3 workgroups and at the 126 of 128 that d = 192 takes; one key; a last
# tile of one key; groups of 32 channels and of all d.
@pytest.mark.parametrize("n_q", [1, 16, 17])
@pytest.mark.parametrize("d,g,n_keys,cap", [
    (256, 32, 1, 3), (256, 256, 31, 3), (256, 32, 97, 3), (256, 256, 192, 3), (256, 32, 193, 3), (256, 256, 384, 3), (256, 32, 385, 3), (256, 32, 769, 3),
    (192, 32, 33, 3), (192, 192, 192, 3), (192, 32, 193, 3), (192, 192, 4064, 128), (192, 32, 8064, 128), (192, 32, 8065, 128),
    (128, 32, 32, 3), (128, 128, 384, 3), (128, 32, 385, 3), (128, 32, 768, 3), (128, 128, 769, 3), (64, 32, 768, 3), (64, 64, 769, 3)])
def test_decode_attention_at_the_edges_of_its_teams(B, d, g, n_q, n_keys, cap):
    test_decode_attention_at_the_edges_of_its_tiles_and_grid(B, d, g, n_q, n_keys, cap, 0.1)


# d = 192: 63 of 64 workgroups scan (252 of 256), and what is left over of the tiles of 32 keys is a second one for a few wavefronts.
# The last size that does not need it, the first and the last that do, and the first of the 64-key tiles.
@pytest.mark.parametrize("n_q", [1, 16, 17])
@pytest.mark.parametrize("g,n_keys,cap", [(32, 16128, 64), (32, 16129, 64), (192, 16384, 64), (32, 16385, 64), (192, 8065, 64), (32, 8192, 64), (32, 32257, 128), (192, 32768, 128)])
def test_decode_attention_of_192_channels_beside_its_whole_grid(B, g, n_q, n_keys, cap):
    test_decode_attention_at_the_edges_of_its_tiles_and_grid(B, 192, g, n_q, n_keys, cap, 0.1)
