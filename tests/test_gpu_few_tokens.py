"""The few-token GEMM (T <= 32) at the edges of its dispatch and tiles, against the oracle: INT32 accumulators
bit-exact, fp16 output within 5e-3 (run with -m gpu on an MI355X)."""
import numpy as np
import pytest

from paper_2310_09259_amd import synth
from tests.util import output_within_tolerance, to_dev, upload

pytestmark = pytest.mark.gpu

# N, K, n_out.  With 256 compute units: one 16-channel block per CU at most (four waves; eight where a row has
# sixteen 128-byte lines), pairs of blocks just above that, single blocks where pairs would leave the busiest CU
# with more (4-bit weights under 8-bit activations: 64 x 64 tiles from 17 tokens on); a last line with one 16-byte
# piece, none and a short fp16 part, ragged N.
SHAPES = [
    (37, 264, 0), (200, 4384, 288), (4096, 296, 24), (4104, 520, 40), (8200, 280, 8),
]


@pytest.mark.parametrize("T", [1, 15, 16, 17, 32])
@pytest.mark.parametrize("N,K,n_out", SHAPES)
@pytest.mark.parametrize("bits,w_bits", [(4, 4), (8, 8), (8, 4)])
def test_few_token_layer(oracle, T, N, K, n_out, bits, w_bits):
    _layer(oracle, T, N, K, n_out, bits, w_bits)


@pytest.mark.parametrize("T", [3, 20])
@pytest.mark.parametrize("bits,w_bits", [(4, 4), (8, 8), (8, 4)])
def test_few_token_layer_whose_weights_are_copied_without_the_read_once_hint(oracle, T, bits, w_bits):
    N, K, n_out = 6500, 8008, 8                      # more than 24 MB, rows that are not whole 128-byte lines
    ldw = (K - n_out) * w_bits // 8
    assert ldw % 128 != 0 and ldw % 16 == 0 and N * ldw > 24 << 20
    _layer(oracle, T, N, K, n_out, bits, w_bits)


@pytest.mark.parametrize("bits,w_bits", [(4, 4), (8, 8), (8, 4)])
def test_few_token_layer_replays_from_a_graph(bits, w_bits):
    """The form with the largest LDS rings (eight waves), captured on first use; eager work between the replays."""
    import torch
    from paper_2310_09259_amd import api
    shp = synth.LayerShape("few_graph", 7, 4384, 200, 288, bits, seed=77, w_bits=0 if w_bits == bits else w_bits)
    d = upload(synth.make_inputs(shp))
    w_red = api.quik_weight_reduce(d["w_q"], d["w_scale"], shp.K_b, w_bits)
    y = torch.zeros((shp.T, shp.N), dtype=torch.float16, device="cuda")
    ws = torch.empty(api.quik_workspace_bytes(shp.T, shp.K, shp.N, shp.n_out, bits), dtype=torch.uint8, device="cuda")
    kept = {"out": y, "workspace": ws}

    def layer(x, **kw):
        if w_bits == bits:
            return api.quik_linear(x, d["idx"], bits, d["w_q"], d["w_scale"], w_red, d["w_out"], **kw)
        return api.quik_linear_w4a8(x, d["idx"], d["w_q"], d["w_scale"], w_red, d["w_out"], **kw)

    x = d["x"].clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer(x, **kept)
    for rep in range(3):
        x.copy_(torch.roll(d["x"], rep, 0))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), layer(x).view(torch.int16)), rep


def _layer(oracle, T, N, K, n_out, bits, w_bits):
    from paper_2310_09259_amd import api
    shp = synth.LayerShape("few", T, K, N, n_out, bits, seed=900 + T + N + K, w_bits=0 if w_bits == bits else w_bits)
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
