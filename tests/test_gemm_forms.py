"""Which kernel and tile the dispatch picks, on 256 compute units (host only, no GPU): the GPU tests that mean to
run a certain form name it by their shapes alone, so the choice for every such shape is pinned here."""
import ctypes as C

import pytest

from paper_2310_09259_amd import api
from tests import test_gpu_few_tokens, test_gpu_parity, test_gpu_tile_rules

CUS = 256
WIDTHS = [(4, 4), (8, 8), (8, 4)]

# (kernel, (rows, cols, waves, groups of waves that split K)); S: 32 x 32 matrix instructions, T: 16 x 16
S64x64, S128x64, S128x128 = (2, (64, 64, 4, 1)), (2, (128, 64, 4, 1)), (2, (128, 128, 4, 1))
S256x192, S192x256 = (2, (256, 192, 8, 1)), (2, (192, 256, 8, 1))
T64x32, T64x64, T64x64_PAIR = (3, (64, 32, 8, 4)), (3, (64, 64, 8, 2)), (3, (64, 64, 4, 1))
T128x64, T128x128, T128x128_K2, T256x128 = (3, (128, 64, 8, 2)), (3, (128, 128, 8, 1)), (3, (128, 128, 8, 2)), (3, (256, 128, 8, 1))


def rows(tokens, channels, waves):
    return 1, (tokens, channels, waves, waves)


def form(T, N, K_b, bits, w_bits):
    return api.quik_debug_gemm_form(T, N, K_b, bits, w_bits, CUS)


TILE_RULES = {                         # shapes of tests/test_gpu_tile_rules.py: 4-bit, 8-bit, 4-bit weights under 8
    (33, 70, 2056, 72): (T64x32, T64x32, T64x32),
    (65, 35, 48, 0): (S64x64, S64x64, T64x64_PAIR),
    (129, 2040, 1880, 24): (T64x32, T64x32, T64x32),
    (100, 8150, 520, 40): (S64x64, S64x64, T64x64_PAIR),
    (100, 8150, 5200, 40): (S64x64, T64x64, T64x64),
    (130, 8190, 4432, 80): (S64x64, T128x64, T128x64),
    (130, 8190, 648, 136): (S64x64, S64x64, T64x64_PAIR),
    (128, 16400, 264, 8): (S128x64, T128x128, S128x64),
    (250, 16300, 264, 8): (S128x128, T128x128, S128x64),
    (500, 16000, 304, 48): (S128x128, S128x128, S128x128),
    (120, 9904, 1032, 128): (S64x64, S64x64, T64x64_PAIR),
    (120, 16472, 1240, 72): (S128x64, T128x128, S128x64),
    (300, 11080, 1240, 40): (S128x128, S128x128, S128x128),
}


def test_tile_rule_shapes_run_the_tiles_they_name():
    assert set(test_gpu_tile_rules.SHAPES) == set(TILE_RULES)
    for (T, N, K, n_out), want in TILE_RULES.items():
        assert tuple(form(T, N, K - n_out, *w) for w in WIDTHS) == want, (T, N, K, n_out)


DEEP = [T64x32, T64x32, T64x32, T64x64, T64x64, T128x64, T128x64, T128x128, T128x128_K2, T256x128, T256x128, T256x128,
        S256x192, S128x128, S128x128, S128x64]


def test_deep_tile_shapes_run_the_tiles_they_name_and_wrap_their_rings():
    assert len(test_gpu_tile_rules.DEEP) == len(DEEP)
    for (T, N, K, n_out, bits, w_bits), want in zip(test_gpu_tile_rules.DEEP, DEEP):
        assert form(T, N, K - n_out, bits, w_bits) == want, (T, N, K, n_out, bits, w_bits)
        stages = -(-(K - n_out) * bits // 1024)            # 128 activation bytes each
        assert stages >= 8 and (want[1][3] == 1 or stages % want[1][3]), (T, N, K, stages)


REPEATS = {                            # layers that test_gpu_parity.py repeats with more workgroups than CUs
    "rep2_64x64": S64x64, "rep2_128x64": S128x64, "rep2_128x128": S128x128, "rep2_64x64_w8a8": S64x64,
    "rep2_128x128_w8a8": S128x128, "rep2_128x64_w4a8": S128x64, "rep2_128x128_w4a8": S128x128,
    "rep2_pair_w8a8": T64x64_PAIR, "rep2_pair_w4a8": T64x64_PAIR, "rep2_rows": (1, (16, 16, 4, 4)),
    "rep2_rows_pairs": (1, (32, 32, 4, 4)), "rep2_rows_w8a8": (1, (16, 16, 4, 4)), "rep2_rows_w4a8": (1, (16, 32, 4, 4)),
}


def test_repeated_layers_have_more_workgroups_than_compute_units():
    shapes = {s.name: s for s in test_gpu_parity.REPEAT_SHAPES if s.name.startswith("rep2_")}
    assert set(shapes) == set(REPEATS)
    for name, s in shapes.items():
        kernel, tile = form(s.T, s.N, s.K_b, s.bits, s.weight_bits)
        assert (kernel, tile) == REPEATS[name], name
        assert -(-s.T // tile[0]) * -(-s.N // tile[1]) > CUS and tile[2] == 4, name


def test_canary_layers_run_the_k_groups_they_name():
    shapes = {s.name: s for s in test_gpu_parity.CANARY_SHAPES}
    for name, want in (("canary_k_groups", T64x32), ("canary_k_groups_w8a8", T128x64)):
        s = shapes[name]
        assert form(s.T, s.N, s.K_b, s.bits, s.bits) == want, name


# The band in which workgroups of four waves, two per CU, are ahead (T, K, N, n_out, w_bits; a 256 x 128 or 128 x 128
# tile per CU took these while the pairs were gone, 5 - 30 % slower)
PAIRS = [
    (512, 4096, 8704, 256, 4), (384, 1024, 24000, 256, 4), (947, 1520, 4232, 256, 4), (333, 1520, 11008, 256, 4),
    (466, 5008, 10880, 328, 4), (1143, 5568, 3648, 712, 4), (1348, 1600, 3264, 256, 4), (120, 1008, 16448, 128, 4),
    (508, 592, 5260, 144, 4), (947, 1520, 4232, 256, 8), (333, 960, 11008, 128, 8), (510, 672, 8384, 168, 8),
    (512, 1536, 8704, 256, 8),
]


def test_few_more_than_one_large_tile_per_cu_run_in_pairs():
    for T, K, N, n_out, w_bits in PAIRS:
        kernel, (rows_, cols, waves, groups) = form(T, N, K - n_out, 8, w_bits)
        assert (kernel, waves, groups) == (2, 4, 1), (T, K, N, n_out, w_bits)


FEW_TOKENS = {                         # shapes of tests/test_gpu_few_tokens.py: channels and waves up to 16 / to 32 tokens
    (37, 264, 0): [((16, 4), (16, 4))] * 3,
    (200, 4384, 288): [((16, 8), (16, 4))] * 3,
    (4096, 296, 24): [((16, 4), (16, 4))] * 3,
    (4104, 520, 40): [((32, 4), (32, 4))] * 3,
    (8200, 280, 8): [((16, 4), (16, 4)), ((16, 4), (16, 4)), ((32, 4), T64x64_PAIR)],
}


def test_few_token_shapes_run_the_forms_they_name():
    assert set(test_gpu_few_tokens.SHAPES) == set(FEW_TOKENS)
    for (N, K, n_out), want in FEW_TOKENS.items():
        for w, (upto16, upto32) in zip(WIDTHS, want):
            for T in (1, 16):
                assert form(T, N, K - n_out, *w) == rows(16, *upto16), (T, N, K, w)
            for T in (17, 32):
                want_form = upto32 if upto32 == T64x64_PAIR else rows(32, *upto32)
                assert form(T, N, K - n_out, *w) == want_form, (T, N, K, w)


def test_layers_without_the_read_once_hint_run_the_few_token_kernel():
    for w in WIDTHS:
        assert form(3, 6500, 8000, *w) == rows(16, 32, 4) and form(20, 6500, 8000, *w) == rows(32, 32, 4), w


def test_wide_w4a8_layers_of_17_to_32_tokens_run_tiles():
    for T in (17, 32):
        assert form(T, 8192, 1024, 8, 4) == rows(32, 32, 4)
        for N, K_b in ((8200, 272), (14464, 832), (18496, 384), (27526, 2032), (24412, 648), (27520, 10752)):
            assert form(T, N, K_b, 8, 4)[0] == 3, (T, N, K_b)
            assert form(T, N, K_b, 8, 8)[0] == form(T, N, K_b, 4, 4)[0] == form(16, N, K_b, 8, 4)[0] == 1, (T, N, K_b)


LINEAR = {                             # layers of tests/test_gpu_parity.py that are there for their tile
    "big_tiles_ragged": S256x192, "big_tiles_w8a8": S128x128, "tiles_192x256": S192x256,
    "tiles_192x256_w8a8_ragged": S192x256, "tiles16_256x128_ragged": T256x128, "tiles16_256x128_w8a8_ragged": S128x128,
    "t32_ragged_n": rows(32, 16, 4), "t5_w8a8": rows(16, 16, 4), "t100": S64x64, "t60_w8a8": S64x64,
}


def test_parity_layers_run_the_tiles_they_name():
    shapes = {s.name: s for s in test_gpu_parity.LINEAR_SHAPES}
    for name, want in LINEAR.items():
        s = shapes[name]
        assert form(s.T, s.N, s.K_b, s.bits, s.bits) == want, name


def test_persistent_kernel_is_reported_where_the_plan_chooses_it():
    for T, N, K_b in ((2048, 11008, 3840), (4096, 28672, 7936), (1024, 15360, 4864), (2048, 4096, 10752), (333, 11008, 3840)):
        choice, plan = api.quik_debug_gemm_plan(T, N, K_b, CUS) or (0, None)
        kernel, tile = form(T, N, K_b, 4, 4)
        assert (kernel == 4) == (choice == 1), (T, N, K_b)
        if kernel == 4:
            assert tile == (256, 32 * plan[2], 8, 1)


@pytest.mark.parametrize("bad", [(0, 8, 64, 4, 4), (4, 0, 64, 4, 4), (4, 8, 0, 4, 4), (4, 8, 63, 4, 4), (4, 8, 64, 4, 8),
                                 (4, 8, 64, 5, 5), (4, 8, 131072, 8, 8)])
def test_form_hook_rejects_what_the_gemm_rejects(bad):
    out = (C.c_int * 4)()
    assert api.load().quik_debug_gemm_form(*bad, CUS, C.cast(out, C.c_void_p)) == -1
    assert api.load().quik_debug_gemm_form(4, 8, 64, 4, 4, CUS, None) == -2
    assert api.load().quik_debug_gemm_form(4, 8, 64, 4, 4, 0, C.cast(out, C.c_void_p)) == -1
