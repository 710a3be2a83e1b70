"""The work this framework is measured on: one QUIK linear layer, called through its public entry points.

A case is one layer of a transformer at one batch of tokens.  The listed ones cover the range a serving process
sees: single-token decode, small and medium batches, prompts of one to four thousand tokens; 4-bit layers on the
dense path, 8-bit layers and 4-bit weights under 8-bit activations for the down-projections that the paper keeps
at 8 bits, the FP6 and the 2:4-sparse forms of the 4-bit layer; odd token counts and ragged widths; two
projections that share their quantized input.

Fields of a case
  T, K, N, n_out   tokens, input features, output features, outlier columns
  form             "int4" | "int8" | "w4a8" | "fp6" | "sp24": which entry points serve the layer
  bias             with a bias or without
  call             "linear"   the layer in one call, on output and workspace buffers the caller keeps
                   "prepared" the same call with its arguments marshalled once (decode loops)
                   "shared"   one quantization, then two GEMMs with different weights on it (gate and up)
"""
import math

import torch

from paper_2310_09259_amd import api

# bits of a quantized activation; bits of a packed weight; bits of a weight as the form's GEMM reads it
X_BITS = {"int4": 4, "int8": 8, "w4a8": 8, "fp6": 4, "sp24": 4}
W_BITS = {"int4": 4, "int8": 8, "w4a8": 4, "fp6": 4, "sp24": 4}
W_STORED = {"int4": 4, "int8": 8, "w4a8": 4, "fp6": 6, "sp24": 4}


def _case(name, T, K, N, n_out, form="int4", bias=False, call="linear"):
    return {"name": name, "T": T, "K": K, "N": N, "n_out": n_out, "form": form, "bias": bias, "call": call}


def listed():
    return [
        # the smallest layer of the configurations: launch and host latency only
        _case("tiny_t16", 16, 512, 512, 32),
        # one sequence being decoded: the weights pass once, the latency of two launches counts
        _case("decode_13b_qkv_t1", 1, 5120, 15360, 256, call="prepared"),
        # sixteen sequences decoded together, down-projection with 4-bit weights under 8-bit activations
        _case("decode_7b_down_w4a8_t16", 16, 11008, 4096, 256, form="w4a8", call="prepared"),
        # a large decode batch, or a short prompt
        _case("batch_13b_qkv_t128", 128, 5120, 15360, 256),
        # a prompt of odd length through gate and up, which share their quantized input
        _case("prompt_7b_gate_up_t333", 333, 4096, 11008, 256, call="shared"),
        # ragged in every direction, with a bias, 8-bit
        _case("ragged_w8a8_t777", 777, 5000, 4090, 104, form="int8", bias=True),
        # 2:4-sparse weights, a prompt of a thousand tokens
        _case("prefill_13b_qkv_sp24_t1024", 1024, 5120, 15360, 256, form="sp24"),
        # the same length on dense weights
        _case("prefill_13b_qkv_t1024", 1024, 5120, 15360, 256),
        # the benchmark's layer
        _case("prefill_7b_up_t2048", 2048, 4096, 11008, 256),
        # the same layer on the FP6 matrix pipe
        _case("prefill_7b_up_fp6_t2048", 2048, 4096, 11008, 256, form="fp6"),
        # the down-projection kept at 8 bits
        _case("prefill_7b_down_w8a8_t2048", 2048, 11008, 4096, 256, form="int8"),
        # the largest layer
        _case("prefill_70b_up_t4096", 4096, 8192, 28672, 256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """T 1 .. 4096, K 512 .. 11008, N 512 .. 28672 over their logarithms, at most the work of the largest listed
    case; widths in steps of 8 (16 columns of every K go with the 4-bit row format), N in steps of 2."""
    while True:
        T = _log_int(rng, 1, 4096)
        K = 16 * _log_int(rng, 32, 688)
        N = 2 * _log_int(rng, 256, 14336)
        if 2 * T * K * N <= 2 * 4096 * 8192 * 28672:
            break
    n_out = min(8 * _log_int(rng, 1, 112), K // 4 // 8 * 8)
    if rng.random() < 0.1:
        n_out = 0
    elif rng.random() < 0.5:
        n_out = min(256, K // 4 // 8 * 8)
    form = rng.choice(("int4", "int4", "int4", "int8", "w4a8", "fp6", "sp24"))
    bias = rng.random() < 0.3
    call = "linear"
    if form == "int4" and rng.random() < 0.2:
        call = "shared"
    elif T <= 64 and rng.random() < 0.5:
        call = "prepared"
    c = _case("", T, K, N, n_out, form, bias, call)
    del c["name"]
    return c


def _rand(gen, shape, dtype=torch.float16, scale=1.0):
    return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * scale).to(dtype)


def _weights(gen, case):
    """One layer's weights: uniform codes, scales U(0.005, 0.02), outlier weights N(0, 0.02); packed for the form."""
    K, N, n_out, form = case["K"], case["N"], case["n_out"], case["form"]
    K_b, bits = K - n_out, W_BITS[form]
    rb = K_b * bits // 8
    ld = (rb + 15) // 16 * 16
    w = {"w_scale": (torch.rand(N, generator=gen, device="cuda") * 0.015 + 0.005).to(torch.float16),
         "w_out": _rand(gen, (N, n_out), scale=0.02) if n_out else None,
         "bias": _rand(gen, (N,), scale=0.5) if case["bias"] else None}
    codes = torch.randint(0, 256, (N, ld), generator=gen, device="cuda", dtype=torch.uint8)
    if form == "sp24":
        # two of every four consecutive columns (two bytes) survive, drawn at random
        keep = torch.tensor([[0xFF, 0x00], [0x0F, 0x0F], [0x0F, 0xF0], [0xF0, 0x0F], [0xF0, 0xF0], [0x00, 0xFF]],
                            dtype=torch.uint8, device="cuda")
        pick = torch.randint(0, 6, (N, ld // 2), generator=gen, device="cuda")
        codes &= keep[pick].reshape(N, ld)
    w["w_reduced"] = api.quik_weight_reduce(codes, w["w_scale"], K_b, bits)
    if form == "fp6":
        w["w_q"] = api.quik_weight_pack_fp6(codes, K_b)
    elif form == "sp24":
        w["w_q"] = api.quik_weight_pack_sp24(codes, K_b, check=False)
    else:
        w["w_q"] = codes
    return w


def prepare(case, seed):
    """Activations N(0, 1) with the outlier columns forty times as large; weights laid out once; the buffers a
    serving loop keeps (output, workspace)."""
    gen = torch.Generator(device="cuda").manual_seed(20231009 + int(seed))
    T, K, N, n_out, form = case["T"], case["K"], case["N"], case["n_out"], case["form"]
    idx = None
    x = torch.randn((T, K), generator=gen, device="cuda", dtype=torch.float32)
    if n_out:
        order = torch.argsort(torch.rand(K, generator=gen, device="cuda"))
        idx = order[:n_out].sort().values.to(torch.int32).contiguous()
        x[:, idx.long()] *= 40.0
    s = {"case": case, "x": x.to(torch.float16), "idx": idx, "w": _weights(gen, case),
         "y": torch.empty((T, N), dtype=torch.float16, device="cuda")}
    if case["call"] == "shared":
        s["w2"] = _weights(gen, case)
        s["y2"] = torch.empty((T, N), dtype=torch.float16, device="cuda")
        ldq = api.quik_packed_row_bytes(K - n_out, 4)
        s["quant"] = (torch.empty((T, ldq), dtype=torch.uint8, device="cuda"),
                      torch.empty(T, dtype=torch.float32, device="cuda"),
                      torch.empty(T, dtype=torch.float32, device="cuda"),
                      torch.empty((T, n_out), dtype=torch.float16, device="cuda"),
                      torch.empty(api.quik_quantize_workspace_bytes(T, 4), dtype=torch.uint8, device="cuda"))
        return s
    if form == "fp6":
        need = api.quik_workspace_bytes_fp6(T, K, N, n_out)
    elif form == "sp24":
        need = api.quik_workspace_bytes_sp24(T, K, N, n_out)
    else:
        need = api.quik_workspace_bytes(T, K, N, n_out, X_BITS[form])
    s["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    if case["call"] == "prepared":
        s["call"], _ = _layer(s, prepared=True)
    return s


def _layer(s, prepared=False):
    form, w = s["case"]["form"], s["w"]
    common = (w["w_q"], w["w_scale"], w["w_reduced"], w["w_out"])
    kept = {"bias": w["bias"], "out": s["y"], "workspace": s["workspace"]}
    if form in ("int4", "int8"):
        fn = api.prepare_linear if prepared else api.quik_linear
        return fn(s["x"], s["idx"], X_BITS[form], *common, **kept)
    if form == "w4a8":
        fn = api.prepare_linear_w4a8 if prepared else api.quik_linear_w4a8
    elif form == "fp6":
        fn = api.prepare_linear_fp6 if prepared else api.quik_linear_fp6
    else:
        fn = api.prepare_linear_sp24 if prepared else api.quik_linear_sp24
    return fn(s["x"], s["idx"], *common, **kept)


def run(state):
    """One pass: the layer's output, or both outputs of the two layers that share their input."""
    call = state["case"]["call"]
    if call == "prepared":
        state["call"]()
        return state["y"]
    if call == "linear":
        return _layer(state)
    K_b = state["case"]["K"] - state["case"]["n_out"]
    xq, scale, zero, x_out, side = api.quik_quantize(state["x"], state["idx"], 4, out=state["quant"])
    for w, y in ((state["w"], state["y"]), (state["w2"], state["y2"])):
        api.quik_gemm_dequant(xq, scale, zero, x_out if state["idx"] is not None else None, K_b, 4, w["w_q"],
                              w["w_scale"], w["w_reduced"], w["w_out"], bias=w["bias"], out=y, workspace=side)
    return state["y"], state["y2"]


def work(case):
    """Bytes: the activations and the stored weights read once, the output written once.  Operations: the integer
    product of the base columns and the fp16 product of the outlier columns."""
    T, K, N, n_out = case["T"], case["K"], case["N"], case["n_out"]
    K_b = K - n_out
    layers = 2 if case["call"] == "shared" else 1
    w_bits = W_STORED[case["form"]]
    per_layer = N * K_b * w_bits // 8 + 2 * N * n_out + 6 * N + (2 * N if case["bias"] else 0) + 2 * T * N
    return {"bytes": 2 * T * K + 4 * n_out + layers * per_layer, "flops": layers * 2 * T * N * K}


def tolerance(case):
    """The integer part is exact, so two correct implementations differ by the order of the fp32 sums of the outlier
    product and hence by single roundings of the fp16 output.  Against the same path in float64 the output's own
    fp16 rounding is what is seen: about 2e-4 in the norm, 4.9e-4 (half an fp16 step) for one element."""
    return {"rel": 8e-4, "max": 2e-3}
