"""Attention with a workgroup per sequence and head (five tiles of 32 keys hold all of them, and there are more sequences than blocks of 64
queries would find room for at once): edges of query groups and key tiles, a fifth query group, fewer queries than keys, infinite values, huge scores."""
import pytest

from tests import test_gpu_glue as glue

pytestmark = pytest.mark.gpu
# batch, queries, keys, heads, head size: 2 (heads of 64: 4) blocks per compute unit and more, for 256 of them
SHAPES = [(17, 1, 160, 32, 128), (17, 33, 33, 32, 128), (9, 65, 65, 32, 128), (9, 96, 97, 32, 128), (9, 97, 128, 32, 128), (7, 128, 129, 40, 128),
          (6, 129, 129, 32, 128), (6, 148, 148, 32, 128), (5, 160, 160, 40, 128), (300, 64, 160, 2, 128), (33, 32, 63, 32, 64), (17, 127, 160, 32, 64),
          (11, 160, 160, 32, 64), (1100, 20, 31, 1, 64)]


@pytest.mark.parametrize("batch,Sq,Sk,H,d", SHAPES)
def test_edges(oracle, batch, Sq, Sk, H, d):
    glue.test_attention_tile_edges(None, oracle, batch, Sq, Sk, H, d)


@pytest.mark.parametrize("spread", [0.5, 30.0])
@pytest.mark.parametrize("batch,Sq,Sk,H,d", [(6, 148, 148, 32, 128), (9, 70, 150, 32, 128), (11, 130, 159, 32, 64), (520, 64, 100, 1, 128)])
def test_infinite_values(batch, Sq, Sk, H, d, spread):
    glue.test_attention_of_infinite_values(None, batch, Sq, Sk, H, d, spread)


@pytest.mark.parametrize("batch,Sq,Sk,H,d", [(6, 148, 148, 32, 128), (11, 130, 159, 32, 64)])
def test_huge_scores(batch, Sq, Sk, H, d):
    glue.test_attention_of_huge_scores(None, batch, Sq, Sk, H, d)
