"""The work that is timed: what a serving program has this library do, over the sizes, formats and directions it does it in.

Every case goes through the public entry points (``binding``, over the C ABI of ``include/srft_kv.h``) with the buffers,
plans and pointer tables that a program keeps between calls.  Kinds:

  write      the write path over one or several plans: ``srft_kv_quantize`` / ``srft_kv_quantize_batched``
  read       the read path over a stored record: ``srft_kv_dequantize`` / ``srft_kv_dequantize_batched``
  attention  one decode step of attention over a stored cache: ``srft_kv_decode_attention``
  scores     scores of queries against stored keys only: ``srft_kv_scores``
  absmax     the statistic lambda is calibrated from: ``srft_kv_channel_absmax``
  cache      the cache manager: a prompt, then decode steps of one token, over buffers the program owns

Stored records are drawn in plain torch (Gaussian values, quantized per group), so a read does not depend on the write path.
"""
from __future__ import annotations

import ctypes as C
import math
import random

import numpy as np
import torch

from paper_2605_05699_amd import binding as B

DEVICE = "cuda"
CHUNK = 1 << 18                     # vectors per step where inputs and 64-bit results are formed


def listed() -> list[dict]:
    w = dict(g=32, bits=4, transform="dft", ragged=False)
    return [
        # the smallest call: two plans of 256 vectors (one layer's K and V of a 256-token prompt): launch latency
        dict(w, name="append_small", kind="write", d=128, plans=2, n=256),
        # one decode step of a batch of 64 sequences with 8 KV heads at d = 96: 512 new vectors for each of 64 plans
        dict(w, name="append_d96", kind="write", d=96, plans=64, n=512),
        # prefill of 4096 tokens, 28 layers x K|V with 2 KV heads: a mid-sized batched write
        dict(w, name="prefill_d128", kind="write", d=128, plans=56, n=8192),
        # bringing back a 4096-token prefix of 26 layers x K|V at d = 256
        dict(w, name="restore_d256", kind="read", d=256, plans=52, n=4096),
        # storing a 131072-token context, 8 KV heads: K and V of two layers
        dict(w, name="store_128k", kind="write", d=128, plans=4, n=1048576),
        # reading that context back
        dict(w, name="read_128k", kind="read", d=128, plans=4, n=1048576),
        # the 8-bit store at the largest head dimension, vector counts that are no multiple of anything, a call per plan
        dict(w, name="store8_d256", kind="write", d=256, plans=1, n=700001, bits=8),
        # reading one plan's prefix of a large serving batch (64 sequences x 8 KV heads x 8192 tokens) at d = 96
        dict(w, name="read_prefix_d96", kind="read", d=96, plans=1, n=4194304),
        # a decode step over a 131072-token context: the 8 query heads of one KV head
        dict(w, name="attention_128k", kind="attention", d=128, n_q=8, n=131072),
        # the same where a step is short: 4 query heads, 4096 tokens, d = 256
        dict(w, name="attention_4k", kind="attention", d=256, n_q=4, n=4096),
        # one batch of a calibration window, odd length
        dict(w, name="calibrate", kind="absmax", d=128, n=1000003),
        # a served sequence pair: prompt of 1000 tokens into 56 plans, then 24 decode steps (the window is flushed on the way)
        dict(w, name="cache_session", kind="cache", d=128, plans=56, n_seq=2, prompt=1000, steps=24),
    ]


def _log_int(rng: random.Random, lo: float, hi: float) -> int:
    return max(1, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _record_bytes(c: dict) -> int:
    return c["d"] * c["bits"] // 8 + 4 * (c["d"] // c["g"])


def draw(rng: random.Random) -> dict:
    kind = rng.choice(["write", "write", "write", "read", "read", "read", "attention", "attention", "scores", "absmax", "cache"])
    d = rng.choice([64, 96, 128, 128, 128, 192, 256, 256] if kind in ("write", "read", "absmax", "cache") else [64, 128, 128, 128, 192, 256])
    if kind in ("write", "read") and rng.random() < 0.1:
        d = rng.choice([32, 160, 224])
    c = dict(kind=kind, d=d, g=32, bits=4, transform="dft", ragged=False)
    if kind in ("write", "read", "cache"):
        c["bits"] = rng.choice([4, 4, 4, 8])
        c["g"] = rng.choice([32, 32, 32, 32, 16, d])
        if kind != "cache" and d & (d - 1) == 0 and rng.random() < 0.1:
            c["transform"] = "hadamard"
    elif kind in ("attention", "scores"):
        c["g"] = rng.choice([32, 32, 32, d])
    per = 2 * d + _record_bytes(c)
    if kind in ("write", "read"):
        c["plans"] = rng.choice([1, 1, 2, _log_int(rng, 2, 100)])
        c["n"] = _log_int(rng, 40, 6e8 / per / c["plans"])
        c["ragged"] = rng.random() < 0.5
    elif kind == "attention":
        c.update(n_q=rng.choice([1, 4, 7, 8, 8, 16, 32]), n=_log_int(rng, 500, 400000))
    elif kind == "scores":
        c.update(n_q=rng.choice([1, 4, 8, 8, 13, 32]), n=_log_int(rng, 500, 1000000))
    elif kind == "absmax":
        c["n"] = _log_int(rng, 2000, 1000000)
    else:
        c.update(plans=rng.choice([2, 32, 56, 64, 80]), n_seq=rng.choice([1, 2, 3, 8]), prompt=_log_int(rng, 30, 800), steps=rng.randint(4, 40))
    return c


# ------------------------------------------------------------------------------------------------------ constants of a plan
def _counts(c: dict) -> list[int]:
    if not c["ragged"]:
        return [c["n"]] * c["plans"]
    return [c["n"] - (37 * i) % (c["n"] // 3 + 1) for i in range(c["plans"])]


def _constants(c: dict, seed: int, plan: int):
    """(sign seed, lambda float32[d], channel gain float32[d]) of one plan."""
    rng = np.random.RandomState((seed * 1009 + plan * 7 + 13) % (2 ** 32))
    lam = np.exp(0.5 * rng.standard_normal(c["d"])).astype(np.float32)
    gain = np.ones(c["d"], dtype=np.float32)
    if plan % 2 == 0:                                          # K: a few persistent outlier channels
        gain[rng.choice(c["d"], size=max(1, c["d"] // 100), replace=False)] = 30.0
    return seed * 1_000_003 + plan, lam, gain


def _plan(c: dict, seed: int, plan: int) -> B.Plan:
    sign_seed, lam, _ = _constants(c, seed, plan)
    return B.Plan(c["d"], c["g"], sign_seed, lam, bits=c["bits"], transform=c["transform"])


def _generator(seed: int, plan: int) -> torch.Generator:
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed * 65537 + plan)
    return g


def _vectors(c: dict, seed: int, plan: int, out: torch.Tensor) -> None:
    """Activations of one plan into out ([n, d] fp16): N(0, 1) times the channel gain."""
    gen, gain = _generator(seed, plan), torch.from_numpy(_constants(c, seed, plan)[2]).to(DEVICE)
    for lo in range(0, out.shape[0], CHUNK):
        part = out[lo:lo + CHUNK]
        part.copy_(torch.randn(part.shape, generator=gen, device=DEVICE) * gain)


def _record(c: dict, seed: int, plan: int, codes: torch.Tensor, scales: torch.Tensor) -> None:
    """A stored record of one plan: Gaussian coefficients, quantized per group."""
    gen, d, g, top = _generator(seed, 1000 + plan), c["d"], c["g"], 7 if c["bits"] == 4 else 127
    for lo in range(0, codes.shape[0], CHUNK):
        k = min(CHUNK, codes.shape[0] - lo)
        w = torch.randn(k, d // g, g, generator=gen, device=DEVICE)
        s = w.abs().amax(dim=2) / top
        q = torch.round(w / s.unsqueeze(2)).to(torch.int16).view(k, d)
        scales[lo:lo + k] = s
        if c["bits"] == 8:
            codes[lo:lo + k] = q.to(torch.int8).view(torch.uint8)
        else:
            codes[lo:lo + k] = ((q[:, 1::2] & 15) * 16 + (q[:, 0::2] & 15)).to(torch.uint8)


def _rows(flat: torch.Tensor, counts: list[int]) -> list[torch.Tensor]:
    return list(torch.split(flat, counts))


# ------------------------------------------------------------------------------------------------------ prepare and run
def prepare(case: dict, seed: int) -> dict:
    return globals()["_prepare_" + {"write": "move", "read": "move", "scores": "attention"}.get(case["kind"], case["kind"])](case, seed)


def _prepare_move(c: dict, seed: int) -> dict:
    counts = _counts(c)
    total = sum(counts)
    plans = [_plan(c, seed, p) for p in range(c["plans"])]
    big = torch.empty(total, c["d"], dtype=torch.float16, device=DEVICE)
    codes = torch.empty(total, c["d"] * c["bits"] // 8, dtype=torch.uint8, device=DEVICE)
    scales = torch.empty(total, c["d"] // c["g"], dtype=torch.float32, device=DEVICE)
    views = [_rows(t, counts) for t in (big, codes, scales)]
    for p in range(c["plans"]):
        if c["kind"] == "write":
            _vectors(c, seed, p, views[0][p])
        else:
            _record(c, seed, p, views[1][p], views[2][p])
    table = B.BatchTable([p.handle for p in plans], *views) if c["plans"] > 1 else None
    return dict(case=c, plans=plans, big=big, codes=codes, scales=scales, table=table)


def _prepare_attention(c: dict, seed: int) -> dict:
    d, n = c["d"], c["n"]
    st = dict(case=c, plans=[_plan(c, seed, p) for p in range(2)])
    st["q"] = torch.randn(c["n_q"], d, generator=_generator(seed, 5000), device=DEVICE).to(torch.float16)
    for p, name in enumerate("kv"):
        st[name] = (torch.empty(n, d // 2, dtype=torch.uint8, device=DEVICE), torch.empty(n, d // c["g"], device=DEVICE))
        _record(c, seed, p, *st[name])
    L, hk, hv = B.lib(), st["plans"][0].handle, st["plans"][1].handle
    if c["kind"] == "scores":
        st["out"] = torch.empty(c["n_q"], n, device=DEVICE)
        need = L.srft_scores_workspace_bytes(hk)
    else:
        st["out"] = torch.empty(c["n_q"], d, device=DEVICE)
        need = L.srft_decode_attention_workspace_bytes(hk, hv, c["n_q"], n)
    st["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEVICE)
    return st


def _prepare_absmax(c: dict, seed: int) -> dict:
    x = torch.empty(c["n"], c["d"], dtype=torch.float16, device=DEVICE)
    _vectors(c, seed, 0, x)
    # the calibration plan has lambda = 1
    return dict(case=c, plans=[B.Plan(c["d"], c["g"], seed * 1_000_003, None)], x=x)


RESIDUAL = 16


def _prepare_cache(c: dict, seed: int) -> dict:
    np_, ns, d = c["plans"], c["n_seq"], c["d"]
    tokens = c["prompt"] + c["steps"]
    pages = -(-tokens // RESIDUAL)
    plans = [_plan(c, seed, p) for p in range(np_)]
    shape = (np_, pages, ns, RESIDUAL)
    st = dict(case=c, plans=plans, capacity=pages * RESIDUAL,
              codes=torch.zeros(*shape, d * c["bits"] // 8, dtype=torch.uint8, device=DEVICE),
              scales=torch.zeros(*shape, d // c["g"], device=DEVICE),
              view=torch.zeros(*shape, d, dtype=torch.float16, device=DEVICE))
    st["prompt"] = torch.empty(np_, ns, c["prompt"], d, dtype=torch.float16, device=DEVICE)
    st["new"] = torch.empty(np_, c["steps"], ns, 1, d, dtype=torch.float16, device=DEVICE)
    for p in range(np_):
        _vectors(c, seed, p, st["prompt"][p].view(-1, d))
        _vectors(c, seed, 7000 + 2 * p, st["new"][p].view(-1, d))
    arr = C.c_void_p * np_
    st["handles"] = arr(*[p.handle for p in plans])
    st["tables"] = [arr(*[t[p].data_ptr() for p in range(np_)]) for t in (st["codes"], st["scales"], st["view"])]
    st["appends"] = [(arr(*[st["prompt"][p].data_ptr() for p in range(np_)]), c["prompt"])]
    st["appends"] += [(arr(*[st["new"][p, s].data_ptr() for p in range(np_)]), 1) for s in range(c["steps"])]
    return st


def run(st: dict):
    return globals()["_run_" + st["case"]["kind"]](st)


def _run_write(st: dict):
    if st["table"] is None:
        B.srft_kv_quantize(st["plans"][0].handle, st["big"], st["codes"], st["scales"])
    else:
        B.srft_kv_quantize_batched(st["table"])
    return st["codes"], st["scales"]


def _run_read(st: dict):
    if st["table"] is None:
        B.srft_kv_dequantize(st["plans"][0].handle, st["codes"], st["scales"], st["big"])
    else:
        B.srft_kv_dequantize_batched(st["table"])
    return st["big"]


def _run_attention(st: dict):
    c = st["case"]
    B.srft_kv_decode_attention(st["plans"][0].handle, st["plans"][1].handle, st["q"], *st["k"], *st["v"],
                               1.0 / math.sqrt(c["d"]), st["out"], st["workspace"])
    return st["out"]


def _run_scores(st: dict):
    B.srft_kv_scores(st["plans"][0].handle, st["q"], *st["k"], st["out"], st["workspace"])
    return st["out"]


def _run_absmax(st: dict):
    return st["plans"][0].channel_absmax(st["x"])


def _run_cache(st: dict):
    # a new conversation over the buffers the program owns (srft_cache_create makes no HIP call)
    c, L, stream = st["case"], B.lib(), torch.cuda.current_stream().cuda_stream
    h = C.c_void_p()
    rc = L.srft_cache_create(C.byref(h), st["handles"], c["plans"], c["n_seq"], st["capacity"], RESIDUAL, *st["tables"])
    for table, t in st["appends"]:
        rc = rc or L.srft_cache_append(h, table, t, stream)
    L.srft_cache_destroy(h)
    if rc:
        raise B.SrftError(rc, "cache")
    return st["codes"], st["scales"], st["view"]


# ------------------------------------------------------------------------------------------------------ work and tolerance
def work(c: dict) -> dict:
    d, rec = c["d"], _record_bytes(c)
    fft = 2.5 * d * math.log2(d)                               # a real FFT; the matrix form does more
    if c["kind"] in ("write", "read"):
        n = sum(_counts(c))
        return dict(bytes=n * (2 * d + rec), flops=n * (fft + 4 * d))
    if c["kind"] == "attention":
        return dict(bytes=2 * c["n"] * rec + c["n_q"] * d * 6, flops=c["n"] * c["n_q"] * (4 * d + 4))
    if c["kind"] == "scores":
        return dict(bytes=c["n"] * (rec + 4 * c["n_q"]) + c["n_q"] * d * 2, flops=c["n"] * c["n_q"] * 2 * d)
    if c["kind"] == "absmax":
        return dict(bytes=c["n"] * 2 * d + 4 * d, flops=c["n"] * (fft + d))
    # every token comes in and is written to the view; a flushed one is stored and its view replaced
    tokens = c["prompt"] + c["steps"]
    n, m = c["plans"] * c["n_seq"] * tokens, c["plans"] * c["n_seq"] * (tokens // RESIDUAL * RESIDUAL)
    return dict(bytes=n * 2 * d + n * 2 * d + m * rec, flops=m * 2 * (fft + 4 * d))


def tolerance(c: dict) -> dict:
    # codes: a value within rounding of a half-integer may fall either way (2-3e-7 of all codes against 64 bits)
    if c["kind"] in ("write", "cache"):
        values = sum(_counts(c)) * c["d"] if c["kind"] == "write" else c["plans"] * c["n_seq"] * (c["prompt"] + c["steps"]) * c["d"]
        differ = max(4e-6 if c["bits"] == 4 else 4e-5, 6.0 / values * (1 if c["bits"] == 4 else 10))
        if c["kind"] == "cache":                               # a code that falls the other way moves its vector's view by one step
            return dict(rel=2e-3, max=0.5, differ=differ)
        return dict(rel=2e-6, max=6e-6, differ=differ)
    if c["kind"] == "read":                                    # fp16 results: now and then the neighbouring value
        return dict(rel=1e-4, max=2e-3)
    if c["kind"] == "absmax":
        return dict(rel=2e-6, max=6e-6)
    return dict(rel=2e-5, max=1e-4)


# ------------------------------------------------------------------------------------------------------ 64-bit results
def _signs(seed: int, d: int) -> np.ndarray:
    """The sign diagonal of a seed: top bits of the splitmix64 stream."""
    m, s, out = 2 ** 64 - 1, seed & (2 ** 64 - 1), []
    for _ in range(d):
        s = (s + 0x9E3779B97F4A7C15) & m
        z = ((s ^ (s >> 30)) * 0xBF58476D1CE4E5B9) & m
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
        out.append(-1.0 if (z ^ (z >> 31)) >> 63 else 1.0)
    return np.array(out)


def _mixing(c: dict) -> np.ndarray:
    """The packed unitary DFT of Eq. 1-2 (or the Walsh-Hadamard matrix) as a d x d matrix."""
    d, h = c["d"], c["d"] // 2
    if c["transform"] == "hadamard":
        k = np.arange(d)
        bits = np.array([[bin(a & b).count("1") for b in k] for a in k])
        return np.where(bits % 2 == 1, -1.0, 1.0) / math.sqrt(d)
    f = np.exp(-2j * math.pi * (np.outer(np.arange(d), np.arange(d)) % d) / d) / math.sqrt(d)
    q = np.empty((d, d))
    q[0], q[h] = f[0].real, f[h].real
    q[1:h], q[h + 1:] = math.sqrt(2) * f[1:h].real, math.sqrt(2) * f[1:h].imag
    return q


def _matrices(c: dict, seed: int, plan: int):
    """(W, R) of one plan in 64 bits, on the GPU: w = W x, x = R (code * scale)."""
    sign_seed, lam, _ = _constants(c, seed, plan)
    if c["kind"] == "absmax":
        sign_seed, lam = seed * 1_000_003, np.ones(c["d"])
    q = _mixing(c) * _signs(sign_seed, c["d"])[None, :]
    lam = lam.astype(np.float64)
    w, r = q * lam[:, None], q.T / np.maximum(lam, 1e-6)[None, :]
    return tuple(torch.from_numpy(np.ascontiguousarray(m)).to(DEVICE) for m in (w, r))


def _decoded(c: dict, codes: torch.Tensor, scales: torch.Tensor) -> torch.Tensor:
    k, d, g = codes.shape[0], c["d"], c["g"]
    if c["bits"] == 8:
        q = codes.view(torch.int8).double()
    else:
        b = codes.to(torch.int32)
        lo, hi = ((b & 15) ^ 8) - 8, ((b >> 4) ^ 8) - 8
        q = torch.stack([lo, hi], dim=2).view(k, d).double()
    return (q.view(k, d // g, g) * scales.double().unsqueeze(2)).view(k, d)


def exact(c: dict, seed: int):
    st = prepare(c, seed)
    top, groups = (7 if c["bits"] == 4 else 127), c["d"] // c["g"]

    def scales_of(x: torch.Tensor, w: torch.Tensor, out: torch.Tensor) -> None:
        for lo in range(0, x.shape[0], CHUNK):
            z = x[lo:lo + CHUNK].double() @ w.t().contiguous()
            out[lo:lo + CHUNK] = z.view(-1, groups, c["g"]).abs().amax(dim=2) / top

    if c["kind"] == "write":
        counts = _counts(c)
        out = torch.empty(sum(counts), groups, dtype=torch.float64, device=DEVICE)
        for p, (x, o) in enumerate(zip(_rows(st["big"], counts), _rows(out, counts))):
            scales_of(x, _matrices(c, seed, p)[0], o)
        return None, out
    if c["kind"] == "read":
        counts = _counts(c)
        out = torch.empty(sum(counts), c["d"], dtype=torch.float64, device=DEVICE)
        for p, (cd, sc, o) in enumerate(zip(_rows(st["codes"], counts), _rows(st["scales"], counts), _rows(out, counts))):
            r = _matrices(c, seed, p)[1].t().contiguous()
            for lo in range(0, cd.shape[0], CHUNK):
                o[lo:lo + CHUNK] = _decoded(c, cd[lo:lo + CHUNK], sc[lo:lo + CHUNK]) @ r
        return out
    if c["kind"] in ("attention", "scores"):
        q = st["q"].double()
        scores = torch.empty(c["n_q"], c["n"], dtype=torch.float64, device=DEVICE)
        rk, rv = _matrices(c, seed, 0)[1].t().contiguous(), _matrices(c, seed, 1)[1].t().contiguous()
        for lo in range(0, c["n"], CHUNK):
            k = _decoded(c, st["k"][0][lo:lo + CHUNK], st["k"][1][lo:lo + CHUNK]) @ rk
            scores[:, lo:lo + CHUNK] = q @ k.t().contiguous()
        if c["kind"] == "scores":
            return scores
        p = torch.softmax(scores / math.sqrt(c["d"]), dim=1)
        out = torch.zeros(c["n_q"], c["d"], dtype=torch.float64, device=DEVICE)
        for lo in range(0, c["n"], CHUNK):
            out += p[:, lo:lo + CHUNK].contiguous() @ (_decoded(c, st["v"][0][lo:lo + CHUNK], st["v"][1][lo:lo + CHUNK]) @ rv)
        return out
    if c["kind"] == "absmax":
        out, w = torch.zeros(c["d"], dtype=torch.float64, device=DEVICE), _matrices(c, seed, 0)[0].t().contiguous()
        for lo in range(0, c["n"], CHUNK):
            out = torch.maximum(out, (st["x"][lo:lo + CHUNK].double() @ w).abs().amax(dim=0))
        return out
    # cache: the scales of the flushed tokens; the view of a flushed token follows its codes, which may fall either way
    np_, ns, d = c["plans"], c["n_seq"], c["d"]
    full = (c["prompt"] + c["steps"]) // RESIDUAL
    out = torch.zeros(st["scales"].shape, dtype=torch.float64, device=DEVICE)
    for p in range(np_):
        new = st["new"][p].view(c["steps"], ns, d).transpose(0, 1)
        x = torch.cat([st["prompt"][p], new], dim=1)[:, :full * RESIDUAL].reshape(ns, full, RESIDUAL, d).transpose(0, 1).reshape(-1, d)
        if x.shape[0]:
            s = torch.empty(x.shape[0], groups, dtype=torch.float64, device=DEVICE)
            scales_of(x, _matrices(c, seed, p)[0], s)
            out[p, :full] = s.view(full, ns, RESIDUAL, groups)
    return None, out, None
