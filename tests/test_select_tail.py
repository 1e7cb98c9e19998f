"""Selection rule where the last picks are made at once (distance 2 by words of 64 tokens on grids of up to 64 columns, distance 1 by index), cut off at every
budget; row lists of ascending and of other index lists."""
import numpy as np
import pytest

from paper_2509_09090_amd import workloads as wl
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from tests import gpu_util
    return gpu_util


def _same(G, oracle, s, gw, gh, k_attn, total, cam=None, radius=0):
    idx, cnt = parity._gpu_select(G, s, gw, gh, k_attn, total, cam, radius)
    want = parity._oracle_select(oracle, s, gw, gh, k_attn, total, cam, radius)
    for b in range(len(s)):
        assert cnt[b] == len(want[b]) and np.array_equal(idx[b, : cnt[b]], want[b]), (b, total)


@pytest.mark.parametrize("gw,gh,k_attn", [(16, 16, 64), (12, 12, 30), (64, 16, 200), (63, 16, 90), (65, 15, 120), (33, 31, 0), (1, 300, 40), (2, 200, 30),
                                          (64, 1, 9), (1024, 1, 200), (5, 13, 1), (32, 32, 256), (3, 3, 2), (1, 1, 0)])
def test_every_budget(G, oracle, gw, gh, k_attn):
    n = gw * gh
    s = wl.scores(4, n, wl.rng_for(101, gw * 1000 + gh, wl.T_SCORES, extra=k_attn))
    s[1] = np.arange(n) % 7                                # the set sampled from: every seventh token, or lines of them
    s[2] = -np.arange(n)                                   # the first rows, the rest of the grid empty
    for total in sorted({k_attn + 1, n // 3, n // 2, n - 1} | ({k_attn, n // 4, (2 * n) // 5, (4 * n) // 5, n} if n < 400 else set())):
        if k_attn <= total <= n:
            _same(G, oracle, s, gw, gh, k_attn, total)


@pytest.mark.parametrize("gw,gh,k_attn,total,radius", [(16, 16, 64, 128, 1), (24, 24, 96, 300, 3), (14, 14, 32, 120, 2)])
def test_around_a_ring(G, oracle, gw, gh, k_attn, total, radius):
    s = wl.scores(16, gw * gh, wl.rng_for(102, gw, wl.T_SCORES))
    _same(G, oracle, s, gw, gh, k_attn, total, wl.cameras(16, gw, gh, 14.0, wl.rng_for(102, gw, wl.T_CAMERA)), radius)


@pytest.mark.parametrize("keep,S,v0,nv", [(1, 5, 2, 3), (128, 276, 0, 256), (255, 276, 20, 256), (256, 300, 10, 256), (257, 700, 3, 600), (1023, 1300, 100, 1024),
                                          (1024, 1300, 276, 1024), (1025, 1400, 7, 1300), (0, 40, 5, 30)])
def test_row_lists(G, keep, S, v0, nv):
    """What the list names and what is not visual, in order of position; places past that stay as they were."""
    import torch
    from paper_2509_09090_amd import binding as B
    rng = np.random.default_rng(keep + S)
    lists = np.stack([np.sort(rng.permutation(nv)[:keep]) for _ in range(6)]).astype(np.int32).reshape(6, keep)
    if keep > 1:
        lists[1] = lists[1][::-1]
        lists[2, keep // 2:] = -1
        lists[3, keep // 2] = lists[3, keep // 2 - 1]
        lists[4, -1] = nv
    per = S - nv + keep
    rows = torch.full((6 * per,), -7, dtype=torch.int32, device="cuda")
    B.sqap_kept_rows(G.to_dev(lists), S, v0, nv, rows)
    want = np.full((6, per), -7, dtype=np.int32)
    for b in range(6):
        named = np.unique(lists[b][(lists[b] >= 0) & (lists[b] < nv)]) + v0
        all_rows = b * S + np.sort(np.concatenate([named, np.arange(v0), np.arange(v0 + nv, S)]))
        want[b, : len(all_rows)] = all_rows
    assert np.array_equal(rows.cpu().numpy().reshape(6, per), want)
