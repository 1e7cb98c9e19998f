"""Infinities and NaN among the values at keys that only the later queries see: those get them, the earlier ones get what the keys that they see give."""
import pytest

pytestmark = pytest.mark.gpu
# batch, queries, keys, heads, head size: every kernel and launch shape (few queries over many keys, blocks of 64, two rounds of them,
# many sequences; small heads)
SHAPES = [(1, 40, 40, 2, 128), (1, 33, 700, 2, 128), (1, 600, 600, 32, 128), (9, 64, 200, 32, 128), (6, 148, 148, 32, 128), (2, 65, 97, 3, 64),
          (1, 300, 331, 4, 64), (2, 70, 100, 3, 32), (1, 33, 90, 2, 16), (1, 2, 2, 1, 128)]


@pytest.mark.parametrize("batch,Sq,Sk,H,d", SHAPES)
def test_values_past_a_query(batch, Sq, Sk, H, d):
    import torch
    from paper_2509_09090_amd import binding as B
    g = torch.Generator().manual_seed(Sq * 7 + Sk + d)
    width, shift, inf = H * d, Sk - Sq, float("inf")
    q, k, v = (torch.randn((batch * n, width), generator=g).half() for n in (Sq, Sk, Sk))
    # (key, column, value): the last key, one that all but the first query see, one in the middle of the queries; both signs in one column
    mid = shift + Sq // 2
    special = [(Sk - 1, 0, inf), (shift + 1, 1, -inf), (mid, d - 1, inf), (Sk - 1, d - 1, -inf), (mid, width - 1, float("nan")), (shift + 1, width - 2, inf)]
    finite = v.clone()
    for b in range(batch):
        for key, column, value in special:
            v[b * Sk + key, column] = value
            finite[b * Sk + key, column] = 0.0
    out = torch.full((batch * Sq, width), 5.0, dtype=torch.float16, device="cuda")
    B.sqap_attention(q.cuda(), k.cuda(), v.cuda(), H, d, out, batch=batch)
    q64, k64, v64 = (t.cuda().double().view(batch, -1, H, d).transpose(1, 2) for t in (q, k, finite))
    s = torch.matmul(q64, k64.transpose(-1, -2).contiguous()) / d ** 0.5
    seen = torch.ones((Sq, Sk), dtype=torch.bool, device="cuda").tril(shift)
    p = torch.softmax(s.masked_fill(~seen, -inf), -1)
    want, size = (torch.matmul(p, t).transpose(1, 2).reshape(batch, Sq, width) for t in (v64, v64.abs()))
    for key, column, value in special:
        want[:, max(0, key - shift):, column] += value
    out = out.double().view(batch, Sq, width)
    usual = want.isfinite()
    assert torch.equal(out.isnan(), want.isnan()) and torch.equal(out[want.isinf()], want[want.isinf()])
    # one half per probability where a column had to be gone through again, 2^-11 of every term; the result's own rounding
    assert torch.all((out - want).abs()[usual] <= (2.0 ** -11 * (size + want.abs()) + 1e-4 * size + 1e-6)[usual])


@pytest.mark.parametrize("batch,Sq,Sk,H,d", [(1, 40, 40, 2, 128), (2, 65, 97, 3, 64), (1, 33, 700, 2, 128)])
def test_infinite_value_without_weight(batch, Sq, Sk, H, d):
    """A key whose score is minus infinity: its infinite value is NaN to the queries that see it, in that column; the rest goes without it."""
    import torch
    from paper_2509_09090_amd import binding as B
    g = torch.Generator().manual_seed(Sq + Sk * 5 + d)
    width, shift, inf = H * d, Sk - Sq, float("inf")
    q, k, v = (torch.randn((batch * n, width), generator=g).half() for n in (Sq, Sk, Sk))
    q[:, 5] = q[:, 5].abs() + 0.5
    key = shift + Sq // 2
    without = k.clone()
    for b in range(batch):
        k[b * Sk + key, 5], v[b * Sk + key, 7] = -inf, inf
        without[b * Sk + key, 5] = -60000.0
    ref_v = torch.where(v.isinf(), torch.zeros_like(v), v)
    out, ref = (torch.full((batch * Sq, width), 5.0, dtype=torch.float16, device="cuda") for _ in range(2))
    B.sqap_attention(q.cuda(), k.cuda(), v.cuda(), H, d, out, batch=batch)
    B.sqap_attention(q.cuda(), without.cuda(), ref_v.cuda(), H, d, ref, batch=batch)
    out, ref = (t.float().view(batch, Sq, width) for t in (out, ref))
    assert torch.all(out[:, Sq // 2:, 7].isnan()) and out.isnan().sum() == batch * (Sq - Sq // 2)
    ok = ~out.isnan()
    assert torch.all((out - ref).abs()[ok] <= (2.0 ** -9 * ref.abs() + 2e-3)[ok])
