"""The native marshalling answers None to every call that is not an ordinary one (host only: no device tensors here), so
that the Python binding serves it as before."""
import pytest
import torch

from paper_2310_09259_amd import api


@pytest.fixture(scope="module")
def call():
    api.load()
    return api._call


def _layer(**kw):
    a = {"kind": 4, "x": torch.zeros((2, 64), dtype=torch.float16), "idx": None, "w": torch.zeros((8, 32), dtype=torch.uint8),
         "sw": torch.zeros(8, dtype=torch.float16), "wr": torch.zeros(16), "wo": None, "bias": None,
         "out": torch.zeros((2, 8), dtype=torch.float16), "ws": torch.zeros(4096, dtype=torch.uint8)}
    a.update(kw)
    return tuple(a.values())


def test_anything_but_plain_device_tensors_goes_to_python(call):
    assert call.linear(*_layer()) is None                                        # host tensors
    assert call.linear(*_layer(x=None)) is None and call.linear(*_layer(x=[1.0])) is None
    assert call.linear(*_layer(kind=4.0)) is None and call.linear(*_layer(kind="4")) is None
    assert call.linear(*_layer(x=torch.zeros((2, 64), dtype=torch.float16, device="meta"))) is None
    assert call.linear(1, 2) is None and call.quantize() is None and call.gemm_dequant(None) is None

    class Sub(torch.Tensor):
        pass
    assert call.linear(*_layer(x=torch.zeros((2, 64), dtype=torch.float16).as_subclass(Sub))) is None


def test_the_binding_still_raises_what_it_raised():
    _, x, idx, w, sw, wr, wo, bias, out, ws = _layer()
    for fn in (lambda: api.quik_linear(x, idx, 4, w, sw, wr, wo, out=out, workspace=ws),
               lambda: api.quik_linear_w4a8(x, idx, w, sw, wr, wo, out=out, workspace=ws),
               lambda: api.quik_linear_fp6(x, idx, w, sw, wr, wo, out=out, workspace=ws),
               lambda: api.quik_linear_sp24(x, idx, w, sw, wr, wo, out=out, workspace=ws),
               lambda: api.quik_quantize(x, idx, 4, out=(w, sw, sw, out, ws)),
               lambda: api.quik_gemm_dequant(w, sw, sw, None, 64, 4, w, sw, wr, wo, out=out, workspace=ws)):
        with pytest.raises(TypeError, match="must be a device tensor"):
            fn()
    with pytest.raises(TypeError):
        api.quik_linear(None, None, 4, w, sw, wr, None, out=out, workspace=ws)


# The marshalling compiled so that host tensors pass for device ones, over stub entry points that answer 0: what it serves,
# refuses and raises, without a GPU.  In a process of its own: a mistake there can take the interpreter down.
HOST_CALLS = r"""
import ctypes as C, importlib.machinery, importlib.util, json, sys, torch
loader = importlib.machinery.ExtensionFileLoader("_quik_call", sys.argv[1])
call = importlib.util.module_from_spec(importlib.util.spec_from_file_location("_quik_call", sys.argv[1], loader=loader))
STUB = C.CFUNCTYPE(C.c_int)(lambda: 0)
call.bind(*[C.cast(STUB, C.c_void_p).value] * 6)
f16, u8, T, K, N, O = torch.float16, torch.uint8, 3, 72, 16, 8

def linear(kind):
    return {"kind": kind, "x": torch.zeros((T, K), dtype=f16), "idx": torch.zeros(O, dtype=torch.int32),
            "w": torch.zeros((1, N, 48) if kind in (6, 24) else (N, 64), dtype=u8), "sw": torch.zeros(N, dtype=f16),
            "wr": torch.zeros(2 * N), "wo": torch.zeros((N, O), dtype=f16), "bias": torch.zeros(N, dtype=f16),
            "out": torch.zeros((T, N), dtype=f16), "ws": torch.zeros(4096, dtype=u8)}

def quantize():
    return {"x": torch.zeros((T, K), dtype=f16), "idx": torch.zeros(O, dtype=torch.int32), "bits": 4,
            "xq": torch.zeros((T, 32), dtype=u8), "scale": torch.zeros(T), "zero": torch.zeros(T),
            "x_out": torch.zeros((T, O), dtype=f16), "ws": torch.zeros(64, dtype=u8)}

def gemm_dequant():
    return {"xq": torch.zeros((T, 32), dtype=u8), "scale": torch.zeros(T), "zero": torch.zeros(T),
            "x_out": torch.zeros((T, O), dtype=f16), "K_b": K - O, "bits": 4, "w": torch.zeros((N, 32), dtype=u8),
            "sw": torch.zeros(N, dtype=f16), "wr": torch.zeros(2 * N), "wo": torch.zeros((N, O), dtype=f16),
            "bias": torch.zeros(N, dtype=f16), "out": torch.zeros((T, N), dtype=f16), "ws": torch.zeros(64, dtype=u8)}

def answer(fn, a):
    try:
        return fn(*a.values())
    except RuntimeError as e:
        return "RuntimeError"

forms = {f"linear {k}": (call.linear, lambda k=k: linear(k)) for k in (4, 8, 84, 6, 24)}
forms["quantize"], forms["gemm_dequant"] = (call.quantize, quantize), (call.gemm_dequant, gemm_dequant)
got = {}
for name, (fn, make) in forms.items():
    got[name + ": plain"] = answer(fn, make())
    for arg, value in make().items():
        if isinstance(value, torch.Tensor):
            a = make()
            torch._C._set_throw_on_mutable_data_ptr(a[arg])
            got[f"{name}: {arg} refuses access"] = answer(fn, a)
            if arg in ("w", "ws") and name != "gemm_dequant":
                continue                                        # bytes
            for dtype in (torch.float64, torch.int64, torch.uint8, torch.float16, torch.int32):
                if dtype != value.dtype and arg not in ("w", "ws", "xq"):
                    got[f"{name}: {arg} of another type, {dtype}"] = answer(fn, {**make(), arg: value.to(dtype)})
            wide = torch.zeros((*value.shape, 2), dtype=value.dtype)[..., 0]       # every other element
            got[f"{name}: {arg} with gaps"] = answer(fn, {**make(), arg: wide})
    a = make()
    for arg in ("idx", "bias"):
        if arg in a:
            got[f"{name}: without {arg}"] = answer(fn, {**a, arg: None, **({"wo": None} if "wo" in a and arg == "idx" else {})})
print(json.dumps(got))
"""


@pytest.fixture(scope="module")
def host_calls(tmp_path_factory):
    import json
    import subprocess
    import sys

    from paper_2310_09259_amd import build
    d = tmp_path_factory.mktemp("host_call")
    src = open(build.CALL_SRC).read()
    for device, host in (("t->is_cuda()", "t->is_cpu()"),
                         ("(void*)c10::hip::getCurrentHIPStream().stream()", "nullptr")):
        assert src.count(device) == 1
        src = src.replace(device, host)
    (d / "call.cpp").write_text(src)
    lib = build.build_call(src=str(d / "call.cpp"), lib=str(d / "_quik_call.so"))
    run = subprocess.run([sys.executable, "-c", HOST_CALLS, lib], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, (run.returncode, run.stderr[-2000:])
    return json.loads(run.stdout)


def test_a_tensor_that_refuses_access_raises(host_calls):
    assert {v for k, v in host_calls.items() if k.endswith(": plain")} == {0}
    refused = {k: v for k, v in host_calls.items() if k.endswith(" refuses access")}
    assert len(refused) == 5 * 9 + 7 + 11
    assert {k: v for k, v in refused.items() if v != "RuntimeError"} == {}


def test_types_and_strides_that_would_be_misread_go_to_python(host_calls):
    other = {k: v for k, v in host_calls.items() if " of another type" in k or k.endswith(" with gaps")}
    assert len(other) > 150 and {k: v for k, v in other.items() if v is not None} == {}
    without = {k: v for k, v in host_calls.items() if ": without " in k}
    assert len(without) == 5 * 2 + 1 + 1 and set(without.values()) == {0}


def test_the_binding_refuses_what_would_be_misread():
    """The ctypes path, before anything is enqueued (host tensors: the message tells the check that was reached)."""
    half, f32 = torch.zeros(8, dtype=torch.float16), torch.zeros(16)
    good = {"outlier_idx": torch.zeros(8, dtype=torch.int32), "w_scale": half, "w_reduced": f32,
            "w_out": torch.zeros((8, 8), dtype=torch.float16), "bias": half, "out": torch.zeros((2, 8), dtype=torch.float16)}
    api._layer_types(*good.values())
    api._layer_types(None, half, f32, None, None, good["out"])
    for nothing in (None, torch.zeros(0, dtype=torch.int64)):                                  # w_out is not read
        api._layer_types(*{**good, "outlier_idx": nothing, "w_out": torch.zeros((8, 8))}.values())
    api._layer_types(*{**good, "w_reduced": torch.zeros(64, dtype=torch.uint8)}.values())      # the raw bytes
    for arg, bad in (("outlier_idx", torch.zeros(8, dtype=torch.int64)), ("w_scale", torch.zeros(8)),
                     ("w_reduced", torch.zeros(16, dtype=torch.float64)), ("w_out", torch.zeros((8, 8))),
                     ("bias", torch.zeros(8)), ("out", torch.zeros((2, 8))), ("out", torch.zeros((2, 8), dtype=torch.uint8))):
        with pytest.raises(TypeError, match=f"{arg} must be "):
            api._layer_types(*{**good, arg: bad}.values())
    for arg, n in (("outlier_idx", 16), ("w_scale", 16), ("w_reduced", 32), ("bias", 16)):
        with pytest.raises(ValueError, match=f"{arg} must be contiguous"):
            api._layer_types(*{**good, arg: torch.zeros(n, dtype=good[arg].dtype)[::2]}.values())


def test_without_the_native_marshalling_calls_go_through_ctypes(monkeypatch, tmp_path):
    api.load()
    monkeypatch.setattr(api, "CALL_PATH", str(tmp_path / "none.so"))
    monkeypatch.setattr(api, "_call", None)
    monkeypatch.setattr(api, "_lib", None)
    with pytest.warns(RuntimeWarning, match="go through ctypes"):
        assert api.quik_version() == 1                                       # the library itself is served
    test_the_binding_still_raises_what_it_raised()


def test_the_library_is_built_where_the_marshalling_cannot_be(monkeypatch, tmp_path, capsys):
    from paper_2310_09259_amd import build
    ran = []

    def run(cmd, **kw):
        ran.append(cmd[0])
        if cmd[0] == "g++":
            raise FileNotFoundError("g++")
    monkeypatch.setattr(build.subprocess, "run", run)
    monkeypatch.setattr(build, "SOURCES", [])
    stale = tmp_path / "_quik_call.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "build_call", lambda *a, _real=build.build_call: _real(*a, lib=str(stale)))
    assert build.build() == build.LIB and ran == [build.HIPCC, "g++"]
    assert "go through ctypes" in capsys.readouterr().err and not stale.exists()


def test_a_marshalling_for_another_torch_is_neither_used_nor_kept(monkeypatch, tmp_path):
    import os
    import shutil

    from paper_2310_09259_amd import build
    api.load()
    src, lib = str(tmp_path / "quik_call.cpp"), str(tmp_path / "_quik_call.so")
    shutil.copy(build.CALL_SRC, src)
    shutil.copy(build.CALL_LIB, lib)
    os.utime(src, (1e9, 1e9))                                                # older than the built one
    assert api._call.BUILT_FOR == build.call_build_stamp()
    ran = []
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **kw: ran.append(cmd))
    build.build_call(incremental=True, src=src, lib=lib)
    assert ran == []                                                         # up to date
    monkeypatch.setattr(build, "call_build_stamp", lambda: "torch 0.0.0, Python 3.0")
    monkeypatch.setattr(api, "_call", None)
    with pytest.warns(RuntimeWarning, match="was built for torch"):
        api._load_call(api._lib)
    assert api._call is api._ThroughCtypes
    build.build_call(incremental=True, src=src, lib=lib)
    assert len(ran) == 1 and ran[0][0] == "g++"
