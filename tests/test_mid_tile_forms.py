"""Which of the 4-bit tiles the estimate picks, on 256 compute units (host only, no GPU)."""
from paper_2310_09259_amd import api
from tests import test_gpu_mid_tiles

T96, T96x128, T128x192 = (3, (96, 96, 4, 1)), (3, (96, 128, 4, 1)), (3, (128, 192, 8, 1))


def form(T, N, K_b):
    return api.quik_debug_gemm_form(T, N, K_b, 4, 4, 256)


def test_shapes_of_the_gpu_test_run_the_tiles_they_name():
    got = [form(T, N, K - n_out) for T, N, K, n_out in test_gpu_mid_tiles.SHAPES]
    assert got[:-1] == [T96, T96, T96x128, T96x128, T128x192, T128x192] and got[-1][0] == 4


def test_measured_shapes_run_the_tile_that_was_ahead():
    for T, K_b, N, want in ((333, 3840, 11008, T96), (92, 7456, 18626, T96), (143, 9976, 20644, T96), (1360, 6984, 1628, T96),
                            (512, 3840, 11008, T128x192), (2325, 5312, 2444, T128x192), (1365, 8296, 5514, (2, (128, 128, 4, 1)))):
        assert form(T, N, K_b) == want, (T, K_b, N)
    for T, K_b, N in ((2445, 2088, 10388), (1945, 3320, 19666), (2048, 3840, 11008), (4096, 7936, 28672), (4096, 4864, 15360)):
        assert form(T, N, K_b)[0] == 4, (T, K_b, N)


def test_shallow_layers_and_small_tiles_keep_their_rule():
    assert form(333, 11008, 1790) == (2, (128, 128, 4, 1))       # fewer than 1792 base columns
    assert form(128, 15360, 4864) == (2, (64, 64, 4, 1))         # up to two 64 x 64 tiles per CU
