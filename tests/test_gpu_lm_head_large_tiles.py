"""The LM head's products in tiles of 256 x 256, at the edges of test_gpu_lm_head_tiles.py and with the masked words of
test_gpu_lm_head_masked_words.py, whose short shapes take tiles of 128 x 128 for every product."""
import numpy as np
import pytest

from tests import test_gpu_lm_head_masked_words as masked
from tests import test_gpu_lm_head_tiles as tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N, d, v, B_s, dh_dtype", [
    (3009, 768, 11009, 4096, "f32"),     # a last word tile of one row, a last k-tile of one word and of one token
    (3073, 768, 11200, 4096, "bf16"),    # a last token tile of one row
    (3072, 768, 11008, 4096, "f32"),     # whole tiles, whole k-tiles
])
def test_edges(lib, N, d, v, B_s, dh_dtype):
    assert [edge for edge, _ in lib.burst_lm_head_tile_plan(lib.lm_head_shape(N, d, v, B_s))] == [256, 256, 256]
    tiles.test_edges(lib, N, d, v, B_s, dh_dtype)


@pytest.fixture
def large(lib, monkeypatch):
    """Logits of more tokens over fewer hidden columns, not split: (max, sum) pairs of 128 words meet in LDS."""
    N, D, V, tile = 1000, 256, 15400, 1024
    assert lib.burst_lm_head_tile_plan(lib.lm_head_shape(N, D, V, tile))[0] == (256, 1)
    for name, value in dict(N=N, D=D, V=V, TILES={"whole": tile}).items():
        monkeypatch.setattr(masked, name, value)
    closed = np.r_[0:8, 5000, 8192:8200, 12032:12160, 14080:14336, V - 8:V]
    monkeypatch.setattr(masked, "CLOSED", closed)


@pytest.mark.parametrize("hidden, weight", [(1.0, -np.inf), (2.0 ** 64, -2.0 ** 66)], ids=["bias of -inf", "overflow"])
def test_words_at_minus_infinity_have_no_share(lib, large, hidden, weight):
    masked.test_words_at_minus_infinity_have_no_share(lib, "whole", hidden, weight)


@pytest.mark.parametrize("closed", [np.r_[8192:8200], np.r_[5000]], ids=["a group", "a word"])
def test_nan_words_reach_the_loss(lib, large, closed):
    masked.test_nan_words_reach_the_loss(lib, "whole", closed)
