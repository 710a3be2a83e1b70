"""Every tile of the FP6 GEMM at its edges: accumulators bit-exact, output within 5e-3 of the oracle and bit-identical to
the int8 path where that does not split K (run with -m gpu)."""
import numpy as np
import pytest

from paper_2310_09259_amd import synth
from tests.util import output_within_tolerance, to_dev, upload

pytestmark = pytest.mark.gpu

# T, N, K, n_out -> tile on 256 compute units (asserted in test_fp6_forms.py): fewer panels than the ring has slots, an
# odd number of panels, a last panel that is not full; one, several and no outlier stages; ragged T and N, with and
# without whole 16-byte output pieces
SHAPES = {
    (12, 74, 184, 16): (64, 64), (70, 136, 2056, 264): (64, 64), (65, 64, 64, 0): (64, 64),
    (97, 8206, 96, 32): (64, 128), (130, 6000, 1104, 48): (64, 128),
    (151, 10910, 176, 40): (128, 128), (300, 7000, 1000, 104): (128, 128),
    (142, 11074, 112, 40): (128, 192), (340, 12000, 1000, 104): (128, 192),
    (709, 8110, 96, 32): (128, 256), (700, 8112, 776, 0): (128, 256),
    (666, 10926, 104, 40): (256, 192), (666, 10928, 904, 136): (256, 192),
    (803, 12438, 112, 40): (256, 256), (770, 14000, 904, 72): (256, 256),
}


# the 64 x 128 tile with eight ring slots (asserted there too): odd and even numbers of panels, none, one and more outlier
# stages than its ring holds
DEEP_RING = [(20, 20098, 4200, 264), (64, 22018, 4104, 8), (33, 19204, 3720, 0)]


# every other tile with nine outlier stages, the last one not full, more than its ring holds at a time
OUTLIER_RING = {
    (40, 2142, 328, 264): (64, 64), (130, 5454, 336, 264): (64, 128), (130, 11072, 408, 264): (128, 128),
    (130, 10986, 328, 264): (128, 192), (400, 12582, 328, 264): (128, 256), (515, 13154, 328, 264): (256, 192),
    (800, 12686, 328, 264): (256, 256),
}


@pytest.mark.parametrize("T,N,K,n_out", [*SHAPES, *OUTLIER_RING, *DEEP_RING])
def test_fp6_tile(oracle, T, N, K, n_out):
    from paper_2310_09259_amd import api
    shp = synth.LayerShape("fp6_tile", T, K, N, n_out, 4, seed=600 + T + N + K)
    inp = synth.make_inputs(shp)
    d = upload(inp)
    b = np.random.default_rng(T).standard_normal(N).astype(np.float16)
    ref = oracle.linear(inp.x, inp.outlier_idx, 4, inp.w_packed, inp.w_scale, inp.w_out, bias=b)
    w_red = api.quik_weight_reduce(d["w_q"], d["w_scale"], shp.K_b, 4)
    w6 = api.quik_weight_pack_fp6(d["w_q"], shp.K_b)
    y = api.quik_linear_fp6(d["x"], d["idx"], w6, d["w_scale"], w_red, d["w_out"], bias=to_dev(b))
    xq6 = api.quik_quantize_fp6(d["x"], d["idx"])[0]
    assert np.array_equal(api.quik_int_gemm_fp6(xq6, w6, shp.K_b).cpu().numpy(), ref.acc)
    ok, worst = output_within_tolerance(y.cpu().numpy(), ref.y)
    assert ok, f"fp16 output outside 5e-3 (worst error / tolerance = {worst:.2f})"
    family, (_, _, _, groups) = api.quik_debug_gemm_form(T, N, shp.K_b, 4, 4, 256)
    if family != 1 and groups == 1:
        y8 = api.quik_linear(d["x"], d["idx"], 4, d["w_q"], d["w_scale"], w_red, d["w_out"], bias=to_dev(b))
        assert np.array_equal(y.cpu().numpy().view(np.uint16), y8.cpu().numpy().view(np.uint16))


def test_fp6_tiles_repeat_bit_identically():
    """More workgroups than compute units, eight calls in a row."""
    import torch
    from paper_2310_09259_amd import api
    for T, N, K, n_out in ((300, 9000, 1000, 104), (90, 20000, 904, 72)):
        shp = synth.LayerShape("fp6_rep", T, K, N, n_out, 4, seed=9)
        d = upload(synth.make_inputs(shp))
        w_red = api.quik_weight_reduce(d["w_q"], d["w_scale"], shp.K_b, 4)
        w6 = api.quik_weight_pack_fp6(d["w_q"], shp.K_b)
        first = None
        for _ in range(8):
            y = api.quik_linear_fp6(d["x"], d["idx"], w6, d["w_scale"], w_red, d["w_out"])
            torch.cuda.synchronize()
            first = y if first is None else first
            assert torch.equal(first.view(torch.int16), y.view(torch.int16))
