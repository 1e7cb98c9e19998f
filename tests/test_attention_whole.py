"""Attention over batches of short whole sequences, more than the device has room for at once: edges of query groups and key tiles, fewer queries
than keys, infinite values, huge scores."""
import pytest

from tests import test_gpu_glue as glue

pytestmark = pytest.mark.gpu
# batch, queries, keys, heads, head size: more than two blocks of 64 queries per compute unit, for 256 of them
SHAPES = [(17, 1, 160, 32, 128), (17, 33, 33, 32, 128), (9, 65, 65, 32, 128), (9, 96, 97, 32, 128), (9, 97, 128, 32, 128), (7, 128, 129, 40, 128),
          (6, 129, 129, 32, 128), (6, 148, 148, 32, 128), (5, 160, 160, 40, 128), (300, 64, 160, 2, 128), (520, 20, 31, 1, 128)]


@pytest.mark.parametrize("batch,Sq,Sk,H,d", SHAPES)
def test_edges(oracle, batch, Sq, Sk, H, d):
    glue.test_attention_tile_edges(None, oracle, batch, Sq, Sk, H, d)


@pytest.mark.parametrize("spread", [0.5, 30.0])
@pytest.mark.parametrize("batch,Sq,Sk,H,d", [(6, 148, 148, 32, 128), (9, 70, 150, 32, 128), (520, 64, 100, 1, 128)])
def test_infinite_values(batch, Sq, Sk, H, d, spread):
    glue.test_attention_of_infinite_values(None, batch, Sq, Sk, H, d, spread)


@pytest.mark.parametrize("batch,Sq,Sk,H,d", [(6, 148, 148, 32, 128), (9, 100, 159, 32, 128)])
def test_huge_scores(batch, Sq, Sk, H, d):
    glue.test_attention_of_huge_scores(None, batch, Sq, Sk, H, d)


@pytest.mark.parametrize("Sq,Sk", [(148, 148), (65, 97), (160, 160), (129, 130)])
def test_the_bits_of_single_calls(Sq, Sk):
    """A sequence of a batch gets what it gets alone, to the bit."""
    import torch
    from paper_2509_09090_amd import binding as B
    g = torch.Generator().manual_seed(Sq + Sk)
    batch, H, d = 9, 32, 128
    q = (1.5 * torch.randn((batch * Sq, H * d), generator=g)).half().cuda()
    kv = torch.randn((batch * Sk, 2 * H * d), generator=g).half().cuda()
    out, alone = torch.empty_like(q), torch.empty_like(q)
    B.sqap_attention(q, kv[:, :H * d], kv[:, H * d:], H, d, out, batch=batch)
    for b in range(batch):
        rows, keys = slice(b * Sq, (b + 1) * Sq), kv[b * Sk:(b + 1) * Sk]
        B.sqap_attention(q[rows], keys[:, :H * d], keys[:, H * d:], H, d, alone[rows])
    assert torch.equal(out.view(torch.int16), alone.view(torch.int16))
