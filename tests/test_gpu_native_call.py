"""The layer calls through the native marshalling (output and workspace given) against the same calls through ctypes: same
bytes, same errors, the caller's stream (run with -m gpu on an MI355X)."""
import pytest

from paper_2310_09259_amd import synth
from tests.util import upload

pytestmark = pytest.mark.gpu

T, K, N, N_OUT = 21, 1040, 200, 48


@pytest.fixture(scope="module")
def layer():
    import torch
    from paper_2310_09259_amd import api
    api.load()
    shp = synth.LayerShape("call", T, K, N, N_OUT, 4, seed=3, sparse24=True)
    d = upload(synth.make_inputs(shp))
    d8 = upload(synth.make_inputs(synth.LayerShape("call8", T, K, N, N_OUT, 8, seed=3)))
    K_b = shp.K_b
    red = api.quik_weight_reduce(d["w_q"], d["w_scale"], K_b, 4)
    red8 = api.quik_weight_reduce(d8["w_q"], d8["w_scale"], K_b, 8)
    w6, w24 = api.quik_weight_pack_fp6(d["w_q"], K_b), api.quik_weight_pack_sp24(d["w_q"], K_b)
    b = torch.randn(N, device="cuda").half()
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    forms = {
        "int4": lambda x, idx, **k: api.quik_linear(x, idx, 4, d["w_q"], d["w_scale"], red, d["w_out"], **k),
        "int8": lambda x, idx, **k: api.quik_linear(x, idx, 8, d8["w_q"], d8["w_scale"], red8, d8["w_out"], **k),
        "w4a8": lambda x, idx, **k: api.quik_linear_w4a8(x, idx, d["w_q"], d["w_scale"], red, d["w_out"], **k),
        "fp6": lambda x, idx, **k: api.quik_linear_fp6(x, idx, w6, d["w_scale"], red, d["w_out"], **k),
        "sp24": lambda x, idx, **k: api.quik_linear_sp24(x, idx, w24, d["w_scale"], red, d["w_out"], **k),
    }
    return api, d, b, ws, forms


@pytest.mark.parametrize("form", ["int4", "int8", "w4a8", "fp6", "sp24"])
def test_native_and_ctypes_calls_agree(layer, form, monkeypatch):
    import torch
    api, d, b, ws, forms = layer
    wide = torch.zeros((T, K + 24), dtype=torch.float16, device="cuda")
    wide[:, :K] = d["x"]
    side = torch.cuda.Stream()
    for x in (d["x"], wide[:, :K], d["x"][3:4]):
        for bias in (None, b):
            want = forms[form](x, d["idx"], bias=bias)                        # no buffers: ctypes
            out = torch.zeros((x.shape[0], N + 8), dtype=torch.float16, device="cuda")[:, :N]
            served = []
            real = api._call.linear
            monkeypatch.setattr(api, "_call", type("Spy", (), {"linear": staticmethod(lambda *a: served.append(real(*a)) or served[-1])}))
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                got = forms[form](x, d["idx"], bias=bias, out=out, workspace=ws)
            monkeypatch.undo()
            torch.cuda.current_stream().wait_stream(side)
            assert served == [0] and got is out
            assert torch.equal(out.contiguous().view(torch.int16), want.view(torch.int16)), (x.shape, bias is None)


def test_native_calls_report_the_library_errors(layer):
    import torch
    api, d, _, ws, forms = layer
    out = torch.zeros((T, N), dtype=torch.float16, device="cuda")
    for form, fn in forms.items():
        with pytest.raises(api.QuikError) as e:
            fn(d["x"], d["idx"], out=out, workspace=ws[:256])
        assert e.value.status == -5, form                                     # workspace too small
        with pytest.raises(api.QuikError) as e:
            fn(d["x"], d["idx"], out=out, workspace=ws[16:])
        assert e.value.status == -3, form                                     # misaligned
        with pytest.raises(TypeError):
            fn(d["x"].float(), d["idx"], out=out, workspace=ws)


def test_native_quantize_and_gemm_agree(layer):
    import torch
    api, d, b, _, _ = layer
    K_b = K - N_OUT
    red = api.quik_weight_reduce(d["w_q"], d["w_scale"], K_b, 4)
    want_q = api.quik_quantize(d["x"], d["idx"], 4)
    bufs = tuple(torch.zeros_like(t) for t in want_q)
    got_q = api.quik_quantize(d["x"], d["idx"], 4, out=bufs)
    assert got_q is bufs and all(torch.equal(g, w) for g, w in zip(got_q, want_q))
    xq, scale, zero, x_out, side = got_q
    args = (xq, scale, zero, x_out, K_b, 4, d["w_q"], d["w_scale"], red, d["w_out"], b)
    want = api.quik_gemm_dequant(*args, workspace=side)
    out = torch.zeros((T, N), dtype=torch.float16, device="cuda")
    assert api.quik_gemm_dequant(*args, out=out, workspace=side) is out
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))
    with pytest.raises(api.QuikError) as e:
        api.quik_gemm_dequant(*args, out=out)                                 # the 4-bit side data is missing
    assert e.value.status == -2


def test_a_tensor_that_refuses_access_raises_as_through_ctypes(layer):
    import torch
    api, d, b, ws, forms = layer
    out = torch.zeros((T, N), dtype=torch.float16, device="cuda")
    for form, fn in forms.items():
        want = fn(d["x"], d["idx"], bias=b)
        for arg in ("x", "idx", "bias", "out", "workspace"):
            a = {"x": d["x"], "idx": d["idx"], "bias": b, "out": out, "workspace": ws}
            a[arg] = a[arg].clone()
            torch._C._set_throw_on_mutable_data_ptr(a[arg])
            for k in ({"out": a["out"], "workspace": a["workspace"]}, {"out": a["out"]}, {"workspace": a["workspace"]}):
                if arg in ("x", "idx", "bias") or arg in k:
                    with pytest.raises(RuntimeError) as e:
                        fn(a["x"], a["idx"], bias=a["bias"], **k)
                    assert not isinstance(e.value, api.QuikError), (form, arg)
        got = fn(d["x"], d["idx"], bias=b, out=out, workspace=ws)                 # and the next call is served
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), form


def test_misread_arguments_are_refused_and_ordinary_ones_without_outliers_served(layer):
    import torch
    api, d, b, ws, forms = layer
    out = torch.zeros((T, N), dtype=torch.float16, device="cuda")
    for form, fn in forms.items():
        for idx, kw in ((d["idx"].long(), {}), (d["idx"], {"bias": b.float()}), (d["idx"], {"out": out.float()})):
            with pytest.raises(TypeError, match="must be torch"):
                fn(d["x"], idx, **{"out": out, "workspace": ws, **kw})
        gaps = torch.stack((d["idx"], d["idx"]), 1)[:, 0]
        with pytest.raises(ValueError, match="outlier_idx must be contiguous"):
            fn(d["x"], gaps, out=out, workspace=ws)
    shp = synth.LayerShape("plain", T, 1024, N, 0, 4, seed=5, sparse24=True)
    p = upload(synth.make_inputs(shp))
    red = api.quik_weight_reduce(p["w_q"], p["w_scale"], shp.K_b, 4)
    w6, w24 = api.quik_weight_pack_fp6(p["w_q"], shp.K_b), api.quik_weight_pack_sp24(p["w_q"], shp.K_b)
    for name, call in (("int4", lambda **k: api.quik_linear(p["x"], None, 4, p["w_q"], p["w_scale"], red, None, **k)),
                       ("w4a8", lambda **k: api.quik_linear_w4a8(p["x"], None, p["w_q"], p["w_scale"], red, None, **k)),
                       ("fp6", lambda **k: api.quik_linear_fp6(p["x"], None, w6, p["w_scale"], red, None, **k)),
                       ("sp24", lambda **k: api.quik_linear_sp24(p["x"], None, w24, p["w_scale"], red, None, **k))):
        want = call()
        assert torch.equal(call(out=out, workspace=ws).view(torch.int16), want.view(torch.int16)), name
