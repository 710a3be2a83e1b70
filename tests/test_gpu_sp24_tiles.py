"""Every tile of the 2:4-sparse GEMM at its edges: accumulators bit-exact, output within 5e-3 of the oracle (run with -m
gpu)."""
import numpy as np
import pytest

from paper_2310_09259_amd import synth
from tests.util import output_within_tolerance, to_dev, upload

pytestmark = pytest.mark.gpu

# T, N, K, n_out -> tile and waves on 256 compute units (asserted in test_sp24_forms.py): fewer panels than the ring has slots, an
# odd number of panels, a last panel that is not full; one, several and no outlier stages; ragged T and N, with and
# without whole 16-byte output pieces
SHAPES = {
    (7, 474, 360, 72): (32, 32, 4), (7, 68, 720, 40): (32, 32, 4), (3, 176, 1112, 0): (32, 32, 4),
    (4, 76, 184, 56): (64, 64, 4), (273, 68, 496, 80): (64, 64, 4), (46, 112, 456, 0): (32, 32, 4),
    (150, 4100, 328, 0): (64, 64, 4),
    (260, 13778, 592, 72): (128, 128, 4), (269, 13640, 864, 0): (128, 128, 4),
    (157, 11164, 96, 40): (128, 128, 8), (132, 10924, 488, 96): (128, 128, 8), (152, 11416, 328, 0): (128, 128, 8),
    (878, 13956, 144, 56): (128, 192, 4), (789, 12388, 448, 48): (128, 192, 4), (811, 12336, 584, 0): (128, 192, 4),
    (257, 13292, 736, 80): (128, 192, 8), (336, 11712, 976, 0): (128, 192, 8),
    (899, 13338, 200, 40): (128, 256, 4), (900, 12292, 432, 40): (128, 256, 4),
    (515, 13810, 304, 40): (256, 192, 8), (529, 13246, 440, 40): (256, 192, 8), (527, 13784, 472, 0): (256, 192, 8),
    (33, 8234, 8456, 264): (64, 32, 4), (64, 8248, 8200, 72): (64, 32, 4), (45, 15362, 5192, 16): (64, 32, 4),
    (44, 15402, 7256, 0): (64, 32, 4),
    (45, 100, 4168, 8): (32, 32, 4), (190, 4098, 2056, 264): (64, 64, 4),
}


# every tile of the general kernel with nine outlier stages, the last one not full: more than its ring holds at a time, so
# that freed slots are refilled with stages that exist
OUTLIER_RING = {
    (33, 4170, 328, 264): (64, 64, 4), (130, 11128, 328, 264): (128, 128, 8), (400, 12308, 528, 264): (128, 128, 4),
    (260, 13062, 1168, 264): (128, 192, 8), (800, 13976, 336, 264): (128, 192, 4), (900, 12298, 328, 264): (128, 256, 4),
    (600, 13096, 528, 264): (256, 192, 8),
}
# the accumulator hook knows no outlier columns and takes another tile for these
OTHER_RAW_TILE = {(257, 13292, 736, 80), (515, 13810, 304, 40)}


@pytest.mark.parametrize("T,N,K,n_out", [*SHAPES, *OUTLIER_RING])
def test_sp24_tile(oracle, T, N, K, n_out):
    from paper_2310_09259_amd import api
    shp = synth.LayerShape("sp24_tile", T, K, N, n_out, 4, seed=700 + T + N + K, sparse24=True)
    inp = synth.make_inputs(shp)
    d = upload(inp)
    b = np.random.default_rng(T).standard_normal(N).astype(np.float16)
    ref = oracle.linear(inp.x, inp.outlier_idx, 4, inp.w_packed, inp.w_scale, inp.w_out, bias=b)
    w_red = api.quik_weight_reduce(d["w_q"], d["w_scale"], shp.K_b, 4)
    w24 = api.quik_weight_pack_sp24(d["w_q"], shp.K_b)
    xq24 = api.quik_quantize_sp24(d["x"], d["idx"])[0]
    assert np.array_equal(api.quik_int_gemm_sp24(xq24, w24, N, shp.K_b).cpu().numpy(), ref.acc)
    for bias in (to_dev(b), None):
        y = api.quik_linear_sp24(d["x"], d["idx"], w24, d["w_scale"], w_red, d["w_out"], bias=bias)
        want = ref.y if bias is not None else oracle.linear(inp.x, inp.outlier_idx, 4, inp.w_packed, inp.w_scale, inp.w_out).y
        ok, worst = output_within_tolerance(y.cpu().numpy(), want)
        assert ok, f"fp16 output outside 5e-3 (worst error / tolerance = {worst:.2f}, bias: {bias is not None})"


def test_sp24_tiles_write_rows_that_are_not_16_byte_aligned():
    """Output rows at an odd stride go element by element: the same bytes, and nothing beyond the row."""
    import torch
    from paper_2310_09259_amd import api
    for T, N, K, n_out in ((273, 68, 496, 80), (157, 11164, 96, 40), (899, 13338, 200, 40)):
        shp = synth.LayerShape("sp24_ld", T, K, N, n_out, 4, seed=11, sparse24=True)
        d = upload(synth.make_inputs(shp))
        w_red = api.quik_weight_reduce(d["w_q"], d["w_scale"], shp.K_b, 4)
        w24 = api.quik_weight_pack_sp24(d["w_q"], shp.K_b)
        want = api.quik_linear_sp24(d["x"], d["idx"], w24, d["w_scale"], w_red, d["w_out"])
        wide = torch.full((T, N + 3), 7.0, dtype=torch.float16, device="cuda")
        api.quik_linear_sp24(d["x"], d["idx"], w24, d["w_scale"], w_red, d["w_out"], out=wide[:, :N])
        assert torch.equal(wide[:, :N].contiguous().view(torch.int16), want.view(torch.int16))
        assert bool((wide[:, N:] == 7.0).all())


def test_sp24_tiles_repeat_bit_identically():
    """More workgroups than compute units, eight calls in a row."""
    import torch
    from paper_2310_09259_amd import api
    for T, N, K, n_out in ((300, 9000, 1000, 104), (90, 20000, 904, 72), (1200, 12000, 520, 40)):
        shp = synth.LayerShape("sp24_rep", T, K, N, n_out, 4, seed=9, sparse24=True)
        d = upload(synth.make_inputs(shp))
        w_red = api.quik_weight_reduce(d["w_q"], d["w_scale"], shp.K_b, 4)
        w24 = api.quik_weight_pack_sp24(d["w_q"], shp.K_b)
        first = None
        for _ in range(8):
            y = api.quik_linear_sp24(d["x"], d["idx"], w24, d["w_scale"], w_red, d["w_out"])
            torch.cuda.synchronize()
            first = y if first is None else first
            assert torch.equal(first.view(torch.int16), y.view(torch.int16))


@pytest.mark.parametrize("T,N,K,n_out", [(9, 1030, 1112, 40), (150, 4100, 328, 72), (157, 11164, 96, 40), (900, 12292, 432, 40)])
def test_sp24_parameters_start_at_any_element(T, N, K, n_out):
    """w_scale and bias at an odd half, scale, zero and w_reduced at an odd float: the same bytes."""
    import torch
    from paper_2310_09259_amd import api
    shp = synth.LayerShape("sp24_odd", T, K, N, n_out, 4, seed=17, sparse24=True)
    d = upload(synth.make_inputs(shp))
    w_red = api.quik_weight_reduce(d["w_q"], d["w_scale"], shp.K_b, 4)
    w24 = api.quik_weight_pack_sp24(d["w_q"], shp.K_b)
    xq, scale, zero, x_out = api.quik_quantize_sp24(d["x"], d["idx"])
    bias = torch.randn(N, device="cuda").half()

    def odd(t):
        out = torch.full((t.numel() + 3,), 9.0, dtype=t.dtype, device="cuda")[1:1 + t.numel()]
        return out.copy_(t)
    want = api.quik_gemm_dequant_sp24(xq, scale, zero, x_out, shp.K_b, w24, d["w_scale"], w_red, d["w_out"], bias=bias)
    got = api.quik_gemm_dequant_sp24(xq, odd(scale), odd(zero), x_out, shp.K_b, w24, odd(d["w_scale"]), odd(w_red), d["w_out"],
                                     bias=odd(bias))
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
