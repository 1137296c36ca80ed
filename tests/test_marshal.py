"""The native marshalling (csrc/host/marshal.cpp) against the calls through ctypes that it stands in front of."""
import array
import ctypes as C
import importlib.util
import shutil
import subprocess
import sys
import sysconfig
from pathlib import Path

import numpy as np
import pytest
import torch

from paper_2605_05699_amd import binding as B
from paper_2605_05699_amd import build as build_module

FAST = ("quantize", "dequantize", "scores", "attention", "absmax", "quantize_batched", "dequantize_batched")


def test_it_is_built():
    assert B._marshal is not None


def test_it_is_named_for_its_interpreter():
    assert B._marshal.__file__ == build_module.LIB_MARSHAL and B._marshal.__file__.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert not (Path(build_module.PKG) / "_marshal.so").exists()


def test_append_takes_what_ctypes_takes():
    native, plain = B.lib().srft_cache_append, C.CDLL(B.LIB_PATH).srft_cache_append
    plain.argtypes, plain.restype = native.argtypes, C.c_int
    arr, cell = (C.c_void_p * 3)(), C.c_void_p()
    for args in ((None, None, 1, None), (cell, arr, 1, 5), (0, 0, 0, 0), (None, arr, -1, cell), (None, C.byref(cell), 1, None), (None, arr, 2 ** 32 + 1, None),
                 (C.c_void_p(None), arr, True, None), (None, None, np.int32(1), None), (None, "x", 1, None), (None, arr, 1.5, None), (None, arr, 1),
                 (2 ** 70, arr, 1, None), (None, arr, None, None)):
        got = []
        for f in (native, plain):
            try:
                got.append(f(*args))
            except Exception as e:
                got.append(type(e))
        assert got[0] == got[1], (args, got)
    assert native.restype is C.c_int and native.argtypes == plain.argtypes


def test_append_is_a_ctypes_function():
    native, plain = B.lib().srft_cache_append, C.CDLL(B.LIB_PATH).srft_cache_append
    assert C.cast(native, C.c_void_p).value == C.cast(plain, C.c_void_p).value
    assert isinstance(native, C._CFuncPtr) and C.sizeof(native) == C.sizeof(plain) and C.addressof(native) and bool(native)
    assert C.c_void_p.from_param(native) is not None and C.byref(native) is not None


def test_what_is_set_on_append_holds_for_its_calls():
    spec = importlib.util.spec_from_file_location(B.__package__ + ".binding_of_its_own", B.__file__)
    own = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(own)
    f = own.lib().srft_cache_append
    assert f(None, None, 1, None) == -1
    f.errcheck = lambda rc, function, args: (rc, function is f, args[2])
    assert f(None, None, 1, None) == (-1, True, 1)
    f.argtypes = [C.c_void_p, C.c_void_p, C.c_double, C.c_void_p]
    assert f(None, None, 1.5, None)[2] == 1.5
    del f.errcheck
    assert f(None, None, 1.5, None) == -1
    assert B.lib().srft_cache_append(None, None, 1, None) == -1                       # (another library object's is as it was)


def test_a_changed_entry_point_does_not_compile(tmp_path):
    """The types of the entry points are the header's: a parameter more in one of them is an error of the compiler."""
    text = (Path(build_module.ROOT) / "include" / "srft_kv.h").read_text()
    changed = text.replace("int srft_kv_channel_absmax(const srft_plan_t* plan, ", "int srft_kv_channel_absmax(const srft_plan_t* plan, int flags, ")
    assert changed != text
    (tmp_path / "srft_kv.h").write_text(changed)
    r = subprocess.run([*build_module._marshal_command(str(tmp_path)), "-fsyntax-only"], capture_output=True, text=True)
    assert r.returncode != 0 and "absmax" in r.stderr and "too few arguments" in r.stderr


def test_the_libraries_are_built_without_a_compiler_for_it(monkeypatch, tmp_path, capsys):
    stale = tmp_path / "_marshal.so"
    stale.write_bytes(b"of other sources")
    monkeypatch.setattr(build_module, "LIB_MARSHAL", str(stale))
    monkeypatch.setattr(build_module.shutil, "which", lambda name: None)
    build_module._marshal(True, False)
    assert not stale.exists() and "g++" in capsys.readouterr().out


def test_the_binding_works_without_it():
    code = """
import sys
sys.modules["paper_2605_05699_amd._marshal"] = None
from paper_2605_05699_amd import binding as B
assert B._marshal is None and B._fast_quantize(1, 2, 3, 4) is None
assert B.lib().srft_cache_append(None, None, 1, None) == -1
"""
    subprocess.run([sys.executable, "-c", code], check=True, cwd=build_module.ROOT)


def test_a_second_library_in_the_process_is_called_through_ctypes(monkeypatch, tmp_path):
    """The native code calls the library it was bound to first; another one's plans never get there."""
    B.lib()
    monkeypatch.setenv("SRFT_KV_LIB", str(shutil.copy(B.LIB_PATH, tmp_path / "other.so")))
    spec = importlib.util.spec_from_file_location(B.__package__ + ".binding_of_another", B.__file__)
    other = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(other)
    address = [C.cast(b.lib().srft_kv_quantize, C.c_void_p).value for b in (B, other)]
    assert address[0] != address[1]
    assert type(other.lib().srft_cache_append) is other.lib()._FuncPtr and type(B.lib().srft_cache_append) is not B.lib()._FuncPtr
    for name in FAST:
        assert getattr(other, "_fast_" + name) is not getattr(other._marshal, name) and getattr(B, "_fast_" + name) is getattr(B._marshal, name)


@pytest.mark.parametrize("args", [("quantize", 4), ("dequantize", 4), ("scores", 6), ("attention", 10), ("absmax", 3)])
def test_what_is_not_on_the_device_is_left_to_the_binding(args):
    name, n = args
    B.lib()
    x = torch.zeros(4, 128, dtype=torch.float16)
    f = getattr(B._marshal, name)
    for a in (x, None, 0, "x", torch.nn.Parameter(x), torch.zeros(2, 2).to_sparse()):
        assert f(1, *([a] * (n - 1))) is None
    assert f() is None and f(*[x] * (n + 1)) is None
    assert B._marshal.quantize_batched(x) is None and B._marshal.dequantize_batched(None) is None


@pytest.mark.gpu
def test_a_table_holds_ctypes_arrays_and_nothing_else():
    """What ctypes refuses for a pointer (a numpy array, a memory view, an array of the standard library) stays refused."""
    table = B.BatchTable([], [], [], [])
    for name in ("plans", "big", "codes", "scales", "n_vec"):
        for wrong in (np.zeros(4, dtype=np.int64), memoryview(bytearray(32)), array.array("q", [0])):
            kept = getattr(table, name)
            setattr(table, name, wrong)
            for f in (B.srft_kv_quantize_batched, B.srft_kv_dequantize_batched):
                with pytest.raises(C.ArgumentError):
                    f(table)
            setattr(table, name, kept)
    B.srft_kv_quantize_batched(table)


@pytest.mark.gpu
@pytest.mark.parametrize("side", [False, True])
def test_results_and_refusals_are_those_of_the_calls_through_ctypes(monkeypatch, side):
    d, n = 128, 77
    p, gen = B.Plan(d, 32, 3), torch.Generator("cuda").manual_seed(1)
    x = torch.randn(n, d, device="cuda", generator=gen).half()
    q = torch.randn(4, d, device="cuda", generator=gen).half()
    ws = torch.empty(B.lib().srft_decode_attention_workspace_bytes(p.handle, p.handle, 4, n), dtype=torch.uint8, device="cuda")

    def empty(*shape, dtype=torch.float32):
        return torch.zeros(*shape, dtype=dtype, device="cuda")

    def calls():
        c, s, back = empty(n, d // 2, dtype=torch.uint8), empty(n, d // 32), empty(n, d, dtype=torch.float16)
        out, sc, m = empty(4, d), empty(4, n), empty(d)
        c2, s2, b2 = torch.zeros_like(c), torch.zeros_like(s), torch.zeros_like(back)
        B.srft_kv_quantize(p.handle, x, c, s)
        B.srft_kv_dequantize(p.handle, c, s, back)
        B.srft_kv_scores(p.handle, q, c, s, sc, ws)
        B.srft_kv_decode_attention(p.handle, p.handle, q, c, s, c, s, 0.1, out, ws)
        B.srft_kv_channel_absmax(p.handle, x, m)
        table = B.BatchTable([p.handle] * 2, [x[:40], x[40:]], [c2[:40], c2[40:]], [s2[:40], s2[40:]])
        B.srft_kv_quantize_batched(table)
        B.srft_kv_dequantize_batched(B.BatchTable([p.handle] * 2, [b2[:40], b2[40:]], [c2[:40], c2[40:]], [s2[:40], s2[40:]]))
        refused = []
        for f, a in ((B.srft_kv_quantize, (p.handle, x.float(), c, s)), (B.srft_kv_quantize, (p.handle, x.t(), c, s)), (B.srft_kv_quantize, (None, x, c, s)),
                     (B.srft_kv_quantize, (p.handle, x.cpu(), c, s)), (B.srft_kv_quantize, (p.handle, x.view(-1)[1:9], c, s)), (B.srft_kv_dequantize, (p.handle, c, s, None)),
                     (B.srft_kv_scores, (p.handle, q, c, s, sc[:, 1:], ws)), (B.srft_kv_scores, (p.handle, q, c, s, sc, ws[:16])),
                     (B.srft_kv_scores, (p.handle, torch.cat([q] * 9), c, s, empty(36, n), ws)),
                     (B.srft_kv_decode_attention, (p.handle, p.handle, q, c, s, c[1:], s, 0.1, out, ws)),
                     (B.srft_kv_decode_attention, (p.handle, p.handle, q, c, s, c, s, float("inf"), out, ws)),
                     (B.srft_kv_decode_attention, (p.handle, p.handle, q, c, s, c, s, 0.1, out, ws[:64])),
                     (B.srft_kv_channel_absmax, (p.handle, x, m[1:])), (B.srft_kv_quantize_batched, (None,))):
            with pytest.raises(Exception) as e:
                f(*a)
            refused.append((e.type, str(e.value)))
        torch.cuda.synchronize()
        return [c, s, back, out, sc, m, c2, s2, b2], refused

    def under():
        if not side:
            return calls()
        with torch.cuda.stream(torch.cuda.Stream()):
            return calls()

    torch.cuda.synchronize()
    got, refused = under()
    for name in FAST:
        assert getattr(B, "_fast_" + name) is getattr(B._marshal, name)
        monkeypatch.setattr(B, "_fast_" + name, lambda *a: None)
    want, also = under()
    assert refused == also
    for a, b in zip(got, want):
        assert torch.equal(a, b) and bool(a.any())
    p.close()
