"""4-bit tiles between 64 x 64 and the 256-row ones (96 x 96 and 96 x 128 in pairs, 128 x 192), and a layer that only the
estimate gives to the persistent kernel: accumulators bit-exact, output within 5e-3 of the oracle (run with -m gpu)."""
import pytest

from tests.test_gpu_tile_rules import _layer

pytestmark = pytest.mark.gpu

# T, N, K, n_out; the tiles on 256 compute units are asserted in test_mid_tile_forms.py.  Ragged in every direction, the
# last integer stage not full, with and without whole 16-byte output pieces.
SHAPES = [(66, 21618, 1992, 144), (450, 9208, 1832, 32), (265, 16726, 1896, 96), (265, 16728, 1888, 0),
          (197, 16454, 1960, 104), (196, 16456, 2056, 24), (261, 21836, 2152, 40)]


@pytest.mark.parametrize("T,N,K,n_out", SHAPES)
def test_mid_tile(oracle, T, N, K, n_out):
    _layer(oracle, T, N, K, n_out, 4, 4)
