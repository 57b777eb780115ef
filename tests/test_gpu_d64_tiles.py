"""Edges of the tiles of the 64-wide heads' kernels: work-groups of 128 query rows with three tiles of 64 rows in LDS.

One row to a row more than a tile on either side, one tile to one more than there are in LDS, waves without rows, the diagonal
of a causal mask through a tile."""
import pytest

from tests.test_gpu_head_layouts import step_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("sq,sk", [(1, 1), (1, 257), (31, 64), (33, 65), (127, 128), (128, 129), (129, 192), (160, 193), (255, 320), (385, 63)])
def test_tiles_of_narrow_heads(lib, sq, sk, causal):
    step_case(lib, 1, 6, 3, 64, sq, sk, causal, 500 + sq + sk, q_pos=40)
