"""GPU parity of the scores-in-the-rotated-domain entry point against the oracle's plain definition."""
import ctypes as C

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


def _tolerance(q, keys_ref64):
    # fp32 accumulation of d terms in the transform of q and in the contraction: about 1e-6 of ||q|| ||k||; the
    # oracle is fp64.  4e-6 leaves room for the two-term fp16 split of q' (about 2^-21 relative per element).
    return 4e-6 * np.linalg.norm(q.astype(np.float64), axis=1)[:, None] * np.linalg.norm(keys_ref64, axis=1)[None, :] + 1e-30


@pytest.mark.parametrize("d", [64, 128, 192, 256])
@pytest.mark.parametrize("n_q,n_keys", [(1, 1), (8, 33), (32, 1000), (5, 4097)])
def test_scores_match_the_definition(B, d, n_q, n_keys):
    g = 32
    keys = W.gaussian_with_outliers(n_keys, d, seed=d + n_keys, outliers=1, gain=15.0)
    q = W.gaussian_with_outliers(n_q, d, seed=7 * d + n_q, outliers=1, gain=4.0)
    lam = W.lognormal_lambda(d, seed=d + 3)
    plan = B.Plan(d, g, 500 + d, lam)
    s = plan.signs
    codes, scales = plan.quantize(torch.from_numpy(keys).cuda())
    got = plan.scores(torch.from_numpy(q).cuda(), codes, scales).cpu().numpy().astype(np.float64)
    c, sc = codes.cpu().numpy(), scales.cpu().numpy()
    ref = O.attention_scores(q, c, sc, s, lam, g)
    back = O.dequantize_f64(c, sc, s, lam, g)
    assert got.shape == (n_q, n_keys)
    assert np.all(np.abs(got - ref) <= _tolerance(q, back)), float((np.abs(got - ref) / _tolerance(q, back)).max())
    # and they are what attention over the dequantized prefix would see, up to that prefix's fp16 rounding
    out = plan.dequantize(codes, scales).cpu().numpy().astype(np.float64)
    via_prefix = q.astype(np.float64) @ out.T
    assert np.all(np.abs(got - via_prefix) <= 2.0 ** -10 * np.abs(q.astype(np.float64)) @ np.abs(out).T + _tolerance(q, back))
    plan.close()


def test_scores_with_wide_groups_hadamard_and_a_grid_cap(B):
    d, n_keys, n_q = 128, 3001, 8
    keys = W.gaussian_with_outliers(n_keys, d, seed=1)
    q = W.gaussian_with_outliers(n_q, d, seed=2)
    for g, transform, form in ((64, "dft", "dense"), (128, "dft", "dense"), (32, "hadamard", "hadamard")):
        lam = W.lognormal_lambda(d, seed=g)
        plan = B.Plan(d, g, 9, lam, transform=transform)
        codes, scales = plan.quantize(torch.from_numpy(keys).cuda())
        qd = torch.from_numpy(q).cuda()
        a = plan.scores(qd, codes, scales)
        B.srft_plan_set_max_workgroups(plan.handle, 3)
        assert torch.equal(a, plan.scores(qd, codes, scales))          # independent of the launch shape
        c, sc = codes.cpu().numpy(), scales.cpu().numpy()
        ref = O.attention_scores(q, c, sc, plan.signs, lam, g, form=form)
        back = O.dequantize_f64(c, sc, plan.signs, lam, g, form=form)
        assert np.all(np.abs(a.cpu().numpy() - ref) <= _tolerance(q, back))
        plan.close()


@pytest.mark.parametrize("d", [64, 128])
def test_every_query_count_and_nothing_written_outside(B, d):
    # n_q = 1..32 walks every kernel instance (16 and 32 rows of queries, every store count) and every partly
    # filled last store; the output sits between two guard zones that must come back untouched.
    g, n_keys, guard = 32, 77, 4096
    keys = W.gaussian_with_outliers(n_keys, d, seed=21, outliers=1, gain=10.0)
    lam = W.lognormal_lambda(d, seed=22)
    plan = B.Plan(d, g, 23, lam)
    codes, scales = plan.quantize(torch.from_numpy(keys).cuda())
    c, sc = codes.cpu().numpy(), scales.cpu().numpy()
    back = O.dequantize_f64(c, sc, plan.signs, lam, g)
    ws = torch.empty(B.lib().srft_scores_workspace_bytes(plan.handle), dtype=torch.uint8, device="cuda")
    for n_q in range(1, 33):
        q = W.gaussian_with_outliers(n_q, d, seed=100 + n_q)
        buf = torch.full((guard + n_q * n_keys + guard,), -12345.0, dtype=torch.float32, device="cuda")
        out = buf[guard:guard + n_q * n_keys].view(n_q, n_keys)
        B.srft_kv_scores(plan.handle, torch.from_numpy(q).cuda(), codes, scales, out, ws)
        torch.cuda.synchronize()
        host = buf.cpu().numpy()
        assert np.all(host[:guard] == -12345.0) and np.all(host[-guard:] == -12345.0), n_q
        got = host[guard:-guard].reshape(n_q, n_keys).astype(np.float64)
        ref = O.attention_scores(q, c, sc, plan.signs, lam, g)
        assert np.all(np.abs(got - ref) <= _tolerance(q, back)), n_q
    plan.close()


@pytest.mark.parametrize("d,transform", [(64, "dft"), (128, "dft"), (192, "dft"), (256, "dft"), (64, "hadamard"), (256, "hadamard")])
@pytest.mark.parametrize("n_q", [1, 9, 16, 17, 32])
def test_every_channel_of_the_transformed_queries(B, d, transform, n_q):
    """Keys with one code of 1 in channel t: the score is channel t of the query's own transform, held to 1e-6 of |q| / lambda_t
    (fp32 butterflies over log2 d levels and the fp16 split: about 2^-21)."""
    lam = W.lognormal_lambda(d, seed=d + 1)
    plan = B.Plan(d, 32, 70 + d, lam, transform=transform)
    t = np.arange(d)
    codes = np.zeros((d, d // 2), dtype=np.uint8)
    codes[t, t // 2] = np.where(t % 2, 16, 1)
    scales = np.ones((d, d // 32), dtype=np.float32)
    q = W.gaussian_with_outliers(n_q, d, seed=n_q + d, outliers=1, gain=4.0)
    q[0] = 0
    q[0, d // 3] = 2.0                                       # an impulse among them
    got = plan.scores(torch.from_numpy(q).cuda(), torch.from_numpy(codes).cuda(), torch.from_numpy(scales).cuda()).cpu().numpy()
    ref = O.attention_scores(q, codes, scales, plan.signs, lam, 32, form="hadamard" if transform == "hadamard" else "dense")
    tol = 1e-6 * np.linalg.norm(q.astype(np.float64), axis=1)[:, None] / lam[None, :].astype(np.float64)
    assert np.all(np.abs(got - ref) <= tol), float((np.abs(got - ref) / tol).max())
    plan.close()


def test_scores_argument_errors(B):
    L = B.lib()
    plan = B.Plan(128, 32, 1)
    q = torch.zeros(4, 128, dtype=torch.float16, device="cuda")
    c = torch.zeros(64, 64, dtype=torch.uint8, device="cuda")
    s = torch.zeros(64, 4, dtype=torch.float32, device="cuda")
    o = torch.zeros(4, 64, dtype=torch.float32, device="cuda")
    ws = torch.zeros(L.srft_scores_workspace_bytes(plan.handle), dtype=torch.uint8, device="cuda")
    args = (q.data_ptr(), 4, c.data_ptr(), s.data_ptr(), 64, o.data_ptr(), ws.data_ptr(), None)
    assert L.srft_kv_scores(plan.handle, *args) == 0
    assert L.srft_kv_scores(None, *args) == -1
    assert L.srft_kv_scores(plan.handle, q.data_ptr(), 0, *args[2:]) == -7
    assert L.srft_kv_scores(plan.handle, q.data_ptr(), 33, *args[2:]) == -7
    assert L.srft_kv_scores(plan.handle, q.data_ptr(), 4, c.data_ptr(), s.data_ptr(), 64, o.data_ptr(), None, None) == -1
    assert L.srft_kv_scores(plan.handle, q.data_ptr(), 4, c.data_ptr(), s.data_ptr(), 0, None, None, None) == 0
    for bad in (B.Plan(96, 32, 1), B.Plan(128, 16, 1), B.Plan(128, 32, 1, bits=8)):
        assert L.srft_kv_scores(bad.handle, *args) in (-2, -3, -9)
        bad.close()
    torch.cuda.synchronize()
    plan.close()


@pytest.mark.parametrize("d,g,n_q,cap", [(64, 32, 16, 2), (64, 64, 17, 1), (128, 32, 17, 2), (128, 128, 3, 1), (192, 32, 32, 1),
                                         (192, 96, 16, 2), (256, 32, 8, 1), (256, 64, 32, 2),
                                         (64, 32, 9, 1), (128, 32, 13, 2), (192, 32, 9, 1), (256, 256, 10, 2), (64, 32, 29, 2)])
def test_scores_at_the_edges_of_tiles_and_of_a_wavefronts_share(B, d, g, n_q, cap):
    """Key counts around one tile and around one, two and three rounds of a capped grid; rows of scores at every alignment
    (odd counts), nothing written past the last one."""
    lam = W.lognormal_lambda(d, seed=d + g)
    plan = B.Plan(d, g, 900 + d, lam)
    n_max = 3200
    keys = W.gaussian_with_outliers(n_max, d, seed=d + 9, outliers=1, gain=15.0)
    q = W.gaussian_with_outliers(n_q, d, seed=d + 10, outliers=1, gain=4.0)
    codes, scales = plan.quantize(torch.from_numpy(keys).cuda())
    c, sc = codes.cpu().numpy(), scales.cpu().numpy()
    ref = O.attention_scores(q, c, sc, plan.signs, lam, g)
    tol = _tolerance(q, O.dequantize_f64(c, sc, plan.signs, lam, g))
    B.srft_plan_set_max_workgroups(plan.handle, cap)
    ws = torch.empty(B.lib().srft_scores_workspace_bytes(plan.handle), dtype=torch.uint8, device="cuda")
    qd = torch.from_numpy(q).cuda()
    for n in (1, 31, 32, 33, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1025, 1537, 3199, 3200):
        flat = torch.full((n_q * n + 64,), -7.0, dtype=torch.float32, device="cuda")
        B.srft_kv_scores(plan.handle, qd, codes[:n].contiguous(), scales[:n].contiguous(), flat[:n_q * n].view(n_q, n), ws)
        torch.cuda.synchronize()
        got = flat.cpu().numpy().astype(np.float64)
        assert np.all(got[n_q * n:] == -7.0), n
        assert np.all(np.abs(got[:n_q * n].reshape(n_q, n) - ref[:, :n]) <= tol[:, :n]), n
    plan.close()
