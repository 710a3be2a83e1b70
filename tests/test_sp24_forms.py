"""Which output tile the 2:4-sparse GEMM picks, on 256 compute units (host only, no GPU)."""
import ctypes as C

from paper_2310_09259_amd import api
from tests import test_gpu_sp24_tiles


def test_shapes_of_the_gpu_test_run_the_tiles_they_name():
    for (T, N, K, n_out), want in {**test_gpu_sp24_tiles.SHAPES, **test_gpu_sp24_tiles.OUTLIER_RING}.items():
        assert api.quik_debug_sp24_form(T, N, K - n_out, n_out, 256) == want, (T, N, K, n_out)
        raw = api.quik_debug_sp24_form(T, N, K - n_out, 0, 256)                  # the accumulator hook's tile
        assert (raw == want) == ((T, N, K, n_out) not in test_gpu_sp24_tiles.OTHER_RAW_TILE), (T, N, K, n_out, raw)
    assert len(set(test_gpu_sp24_tiles.SHAPES.values())) == 9


def test_measured_shapes_run_the_tile_that_was_ahead():
    for T, N, K, n_out, want in ((1024, 15360, 5120, 256, (128, 256, 4)), (1398, 4672, 9312, 56, (128, 128, 4)),
                                 (333, 11008, 4096, 256, (128, 192, 8)), (16, 4096, 4096, 256, (32, 32, 4)),
                                 (3526, 2592, 9440, 80, (256, 192, 8)), (128, 15360, 5120, 256, (64, 64, 4)),
                                 (50, 15968, 5600, 24, (64, 32, 4)), (64, 15360, 5120, 256, (64, 32, 4))):
        assert api.quik_debug_sp24_form(T, N, K - n_out, n_out, 256) == want, (T, N, K, n_out)


def test_form_hook_rejects_what_the_gemm_rejects():
    out = (C.c_int * 3)()
    for bad in ((0, 8, 64, 0, 256), (4, 0, 64, 0, 256), (4, 8, 0, 0, 256), (4, 8, 131072, 0, 256), (4, 8, 64, -1, 256), (4, 8, 64, 0, 0)):
        assert api.load().quik_debug_sp24_form(*bad, C.cast(out, C.c_void_p)) == -1
    assert api.load().quik_debug_sp24_form(4, 8, 64, 0, 256, None) == -2
