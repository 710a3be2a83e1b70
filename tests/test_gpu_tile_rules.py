"""Every tile that the per-tile GEMM's rules can choose between one tile and one round, at its edges, against the
oracle: INT32 accumulators bit-exact, fp16 output within 5e-3 (run with -m gpu on an MI355X)."""
import numpy as np
import pytest

from paper_2310_09259_amd import synth
from tests.util import output_within_tolerance, to_dev, upload

pytestmark = pytest.mark.gpu

# T, N, K, n_out.  The tiles they run on 256 compute units, for 4 / 8 / 4-under-8 bits, are asserted in
# test_gemm_forms.py (S: 32 x 32 matrix instructions, T: 16 x 16, P: two workgroups per CU):
SHAPES = [
    (33, 70, 2056, 72),       # T 64 x 32 for all; eight and sixteen integer stages, the last not full, two outlier stages
    (65, 35, 48, 0),          # S / S / T 64 x 64 P: one stage, no outlier columns
    (129, 2040, 1880, 24),    # T 64 x 32 for all, ragged in both directions, one short outlier stage
    (100, 8150, 520, 40),     # S / S / T 64 x 64 P
    (100, 8150, 5200, 40),    # S 64 x 64 P / T 64 x 64 / T 64 x 64
    (130, 8190, 4432, 80),    # S 64 x 64 P / T 128 x 64 / T 128 x 64
    (130, 8190, 648, 136),    # S / S / T 64 x 64 P
    (128, 16400, 264, 8),     # S 128 x 64 P / T 128 x 128 / S 128 x 64 P
    (250, 16300, 264, 8),     # S 128 x 128 P / T 128 x 128 / S 128 x 64 P
    (500, 16000, 304, 48),    # S 128 x 128 P for all
    (120, 9904, 1032, 128),   # S / S / T 64 x 64 P: whole 16-byte output pieces, more stages than the ring has
    (120, 16472, 1240, 72),   # S 128 x 64 P / T 128 x 128 / S 128 x 64 P: the same
    (300, 11080, 1240, 40),   # S 128 x 128 P for all: the same
]


# T, N, K, n_out, bits, w_bits: enough integer stages for the ring to wrap inside the unguarded loop (an odd number
# with K groups, so that the groups differ), ragged T and last stage, several outlier stages; N whole 16-byte output
# pieces or not.  The tiles are asserted in test_gemm_forms.py.
DEEP = [
    (33, 72, 2256, 72, 8, 8), (33, 72, 2256, 72, 8, 4), (129, 2044, 2256, 72, 4, 4),          # T 64 x 32, four groups
    (100, 8152, 5288, 136, 8, 8), (100, 8152, 5288, 136, 8, 4),                               # T 64 x 64, two groups
    (130, 8192, 4368, 152, 8, 8), (66, 8442, 2264, 104, 8, 4),                                # T 128 x 64, two groups
    (73, 18504, 1240, 72, 8, 8), (73, 18010, 3104, 272, 8, 4),                                # T 128 x 128, one / two groups
    (201, 18406, 1432, 136, 8, 8), (389, 14616, 1176, 136, 8, 4), (389, 14614, 1176, 136, 8, 4),   # T 256 x 128
    (387, 16440, 1112, 80, 8, 8),                                                             # S 256 x 192
    (300, 11082, 1368, 168, 8, 8), (300, 11082, 1368, 168, 8, 4), (120, 16470, 1368, 168, 8, 4),   # S in pairs
]


@pytest.mark.parametrize("T,N,K,n_out,bits,w_bits", DEEP)
def test_tile_with_many_stages(oracle, T, N, K, n_out, bits, w_bits):
    _layer(oracle, T, N, K, n_out, bits, w_bits)


@pytest.mark.parametrize("T,N,K,n_out", SHAPES)
@pytest.mark.parametrize("bits,w_bits", [(4, 4), (8, 8), (8, 4)])
def test_tile_of_the_rules(oracle, T, N, K, n_out, bits, w_bits):
    _layer(oracle, T, N, K, n_out, bits, w_bits)


def _layer(oracle, T, N, K, n_out, bits, w_bits):
    from paper_2310_09259_amd import api
    shp = synth.LayerShape("tile", T, K, N, n_out, bits, seed=700 + T + N + K, w_bits=0 if w_bits == bits else w_bits)
    inp = synth.make_inputs(shp)
    d = upload(inp)
    b = np.random.default_rng(T).standard_normal(N).astype(np.float16)
    ref = oracle.linear(inp.x, inp.outlier_idx, bits, inp.w_packed, inp.w_scale, inp.w_out, bias=b, w_bits=w_bits)
    w_red = api.quik_weight_reduce(d["w_q"], d["w_scale"], shp.K_b, w_bits)
    xq, scale, zero, x_out, side = api.quik_quantize(d["x"], d["idx"], bits)
    if w_bits == bits:
        y = api.quik_linear(d["x"], d["idx"], bits, d["w_q"], d["w_scale"], w_red, d["w_out"], bias=to_dev(b))
        accs = [api.quik_debug_int_gemm(xq, d["w_q"], shp.K_b, bits)]
        if bits == 4:
            accs.append(api.quik_debug_int_gemm(xq, d["w_q"], shp.K_b, 4, workspace=side, w_reduced=w_red))
    else:
        y = api.quik_linear_w4a8(d["x"], d["idx"], d["w_q"], d["w_scale"], w_red, d["w_out"], bias=to_dev(b))
        accs = [api.quik_int_gemm_w4a8(xq, d["w_q"], shp.K_b)]
    for acc in accs:
        assert np.array_equal(acc.cpu().numpy(), ref.acc)
    ok, worst = output_within_tolerance(y.cpu().numpy(), ref.y)
    assert ok, f"fp16 output outside 5e-3 (worst error / tolerance = {worst:.2f})"
