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
