"""Scales of rows whose largest value is a binary32 value and no half: rotated rows and folded weight rows.  The scale takes two roundings, the quotient by 7
to binary32 and that to half; ties between two halves that the first one makes or breaks are met by one rotated row in 24 500 and one folded row in
660, so there are many rows here."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from tests import gpu_util
    return gpu_util


def _same(got, want):
    codes, scales = got
    assert np.array_equal(np.asarray(scales).view(np.uint16), np.asarray(want[1]).view(np.uint16))
    assert np.array_equal(codes, want[0])


def _folded(G, W, c, flags=0):
    import torch
    from paper_2509_09090_amd import binding as B
    q = torch.zeros((W.shape[0], W.shape[1] // 2), dtype=torch.uint8, device="cuda")
    s = torch.zeros((W.shape[0],), dtype=torch.float16, device="cuda")
    B.sqap_quantize_weight_folded(G.to_dev(W), G.to_dev(c), q, s, flags)
    torch.cuda.synchronize()
    return q.cpu().numpy(), s.cpu().numpy()


def test_folded_rows_at_ties(G, oracle):
    """One value per row, a channel each: the product of two halves is the row's largest value."""
    pairs = [(0x2401, 0x3d40), (0x2402, 0x3e20), (0x2404, 0x3cd0)]
    W, c = np.zeros((len(pairs), 64), np.float16), np.ones(64, np.float16)
    for i, (w, scale) in enumerate(pairs):
        W[i, 5 * i] = np.uint16(w).view(np.float16)
        c[5 * i] = np.uint16(scale).view(np.float16)
    want = oracle.quantize_rows_folded(W, c)
    assert want[1][0].view(np.uint16) == 0x1a02                     # by definition, one rounding would make it 0x1a01
    _same(_folded(G, W, c), want)


@pytest.mark.parametrize("N,K", [(60000, 64), (12000, 2048), (3000, 11008)])
def test_folded_rows(G, oracle, N, K):
    """A value in every row, at a place of its own, and a smaller one."""
    rng = np.random.default_rng(K)
    W, at, place = np.zeros((N, K), np.float16), np.arange(N), rng.integers(K, size=N)
    W[at, place] = (0.02 * rng.standard_normal(N)).astype(np.float16)
    W[at, (place + 9) % K] = W[at, place] * np.float16(0.125)
    c = (np.abs(rng.standard_normal(K)) + 0.01).astype(np.float16)
    _same(_folded(G, W, c), oracle.quantize_rows_folded(W, c))


@pytest.mark.parametrize("K", [64, 192, 1024])
@pytest.mark.parametrize("weight", [False, True])
def test_rotated_rows_of_every_half(G, oracle, K, weight):
    """Every finite half alone in a row, rotated: its quotient by the square root of the block."""
    halves = np.arange(1, 0x7c00, dtype=np.uint16).view(np.float16)
    if K > 192:
        halves = halves[::7]
    X = np.zeros((len(halves), K), np.float16)
    X[np.arange(len(halves)), np.arange(len(halves)) % K] = halves
    want = oracle.quantize_rows(X, rotate=True)
    _same(G.gpu_quantize(X, rotate=True, weight=weight), want)


def test_rotated_rows_after_the_norm(G, oracle):
    import torch
    from paper_2509_09090_amd import binding as B
    rng = np.random.default_rng(5)
    X = rng.standard_normal((60000, 64), dtype=np.float32).astype(np.float16)
    gamma = (1 + 0.1 * rng.standard_normal(64)).astype(np.float16)
    _, y = oracle.rmsnorm_rows(X, gamma, 1e-5)
    want = oracle.quantize_rows(y, rotate=True)
    q = torch.zeros((len(X), 32), dtype=torch.uint8, device="cuda")
    s = torch.zeros((len(X),), dtype=torch.float16, device="cuda")
    B.sqap_rmsnorm_quantize_act(G.to_dev(X), None, G.to_dev(gamma), 1e-5, q, s, flags=B.ROTATE_HADAMARD)
    torch.cuda.synchronize()
    _same((q.cpu().numpy(), s.cpu().numpy()), want)
