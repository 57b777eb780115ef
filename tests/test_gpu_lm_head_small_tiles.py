"""The LM head's products in tiles of 128 x 128 and of 256 x 256 (lm_plan) at the edges of either: a tile of one token or word, a last
tile of 128 words that is not there (an odd number of them in the padded vocabulary), one and two k-tiles, and shapes large enough for the
large tiles, ragged in all three directions."""
import pytest

from tests import test_gpu_lm_head_tiles as tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N, d, v, B_s, dh_dtype", [
    (127, 256, 128, 256, "f32"),       # one tile of words of two
    (128, 512, 129, 256, "bf16"),      # the second one of one word
    (129, 256, 257, 256, "f32"),       # three of four, a token tile of one row
    (385, 768, 1000, 512, "bf16"),     # four token tiles, the last of one row
    (250, 1024, 8191, 1024, "f32"),    # the vocabulary in parts
    (1000, 256, 15361, 1024, "f32"),   # large tiles for the logits
    (1025, 1024, 14337, 2048, "bf16"), # large tiles for both gradients
])
def test_edges_of_either_tile(lib, N, d, v, B_s, dh_dtype):
    tiles.test_edges(lib, N, d, v, B_s, dh_dtype)
