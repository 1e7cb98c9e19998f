"""Decode attention over caches long enough that more workgroups than attend are launched (they only touch cache lines): the output, the cache
row and the codes for head counts with all of a head's workgroups on one XCD, on two, and with no or few compute units to spare."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("H,d,past", [(8, 128, 575), (8, 128, 576), (32, 128, 577), (4, 128, 700), (12, 128, 640), (2, 128, 600),
                                      (64, 128, 600), (16, 64, 1300), (8, 8, 900), (24, 96, 601), (120, 64, 590)])
def test_decode_attention_with_helpers(G, oracle, H, d, past):
    import torch
    from paper_2509_09090_amd import binding as B
    rng = np.random.default_rng(H + d + past)
    width = H * d
    QKV = rng.standard_normal((1, 3 * width)).astype(np.float16)
    prefix = rng.standard_normal((past, 2 * width)).astype(np.float16)
    pos = np.array([past], dtype=np.int32)
    q_rot = oracle.rope(QKV[:, :width].reshape(1, H, d), pos)
    k_rot = oracle.rope(QKV[:, width:2 * width].reshape(1, H, d), pos)
    keys = np.concatenate([prefix[:, :width].reshape(past, H, d), k_rot])
    values = np.concatenate([prefix[:, width:].reshape(past, H, d), QKV[:, 2 * width:].reshape(1, H, d)])
    want = oracle.attention(q_rot, keys, values).reshape(1, width)
    cache = torch.full((past + 1, 2 * width + 8), 3.0, dtype=torch.float16, device="cuda")       # rows that do not begin with a line
    cache[:past, :2 * width] = G.to_dev(prefix)
    quantize = width <= 8192
    O = torch.full((1, width), float("nan"), dtype=torch.float16, device="cuda")
    Xq = torch.zeros((1, width // 2), dtype=torch.uint8, device="cuda") if quantize else None
    sx = torch.zeros((1,), dtype=torch.float16, device="cuda") if quantize else None
    counter = torch.zeros((1,), dtype=torch.int32, device="cuda") if quantize else None
    B.sqap_decode_attention(G.to_dev(QKV), G.to_dev(pos), H, d, cache[:, :2 * width], past, O, Xq, sx, counter)
    torch.cuda.synchronize()
    assert G.assert_fp16_close(O.cpu().numpy(), want) >= 0
    row = cache[past].cpu().numpy()
    assert G.assert_fp16_close(row[None, :width], k_rot.reshape(1, width)) <= width // 100
    assert np.array_equal(row[width:2 * width].view(np.uint16), QKV[0, 2 * width:].view(np.uint16)) and np.all(row[2 * width:] == 3.0)
    assert np.array_equal(cache[:past, :2 * width].cpu().numpy().view(np.uint16), prefix.view(np.uint16))
    if quantize:
        assert int(counter.item()) == 0
        q2, s2 = torch.empty_like(Xq), torch.empty_like(sx)
        B.sqap_quantize_act(O, None, q2, s2)
        torch.cuda.synchronize()
        assert torch.equal(q2, Xq) and torch.equal(s2.view(torch.int16), sx.view(torch.int16))
