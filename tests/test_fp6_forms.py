"""Which output tile the FP6 GEMM picks, on 256 compute units (host only, no GPU)."""
import ctypes as C

from paper_2310_09259_amd import api
from tests import test_gpu_fp6_tiles


def test_shapes_of_the_gpu_test_run_the_tiles_they_name():
    for (T, N, K, n_out), want in {**test_gpu_fp6_tiles.SHAPES, **test_gpu_fp6_tiles.OUTLIER_RING}.items():
        assert api.quik_debug_fp6_form(T, N, K - n_out, 256) == want, (T, N, K, n_out)


def test_measured_shapes_run_the_tile_that_was_ahead():
    for T, N, K_b, want in ((2048, 11008, 3840, (256, 192)), (4096, 28672, 7936, (256, 256)), (1024, 15360, 4864, (256, 256)),
                            (2048, 4096, 10752, (128, 256)), (333, 11008, 3840, (128, 192)), (16, 4096, 3840, (64, 64))):
        assert api.quik_debug_fp6_form(T, N, K_b, 256) == want, (T, N, K_b)


def test_large_layers_of_few_tokens_run_the_deep_ring():
    for T, N, K, n_out in test_gpu_fp6_tiles.DEEP_RING:
        assert api.quik_debug_fp6_slots(T, N, K - n_out, 256) == 8, (T, N, K, n_out)
        assert api.quik_debug_fp6_form(T, N, K - n_out, 256) == (64, 128)
    for T, N, K_b in ((65, 19600, 7128), (16, 4096, 3840), (60, 11008, 3840), (2048, 11008, 3840)):
        assert api.quik_debug_fp6_slots(T, N, K_b, 256) == 6, (T, N, K_b)
    for bad in ((0, 8, 64, 256), (4, 0, 64, 256), (4, 8, 0, 256), (4, 8, 131072, 256), (4, 8, 64, 0)):
        assert api.load().quik_debug_fp6_slots(*bad) == -1


def test_form_hook_rejects_what_the_gemm_rejects():
    out = (C.c_int * 2)()
    for bad in ((0, 8, 64, 256), (4, 0, 64, 256), (4, 8, 0, 256), (4, 8, 131072, 256), (4, 8, 64, 0)):
        assert api.load().quik_debug_fp6_form(*bad, C.cast(out, C.c_void_p)) == -1
    assert api.load().quik_debug_fp6_form(4, 8, 64, 256, None) == -2
