"""Rows whose RMSNorm factor lies so close to the middle between two binary32 values that the device's estimate leaves it open and the exact
sum of squares has to decide (quant_math.h: norm_factor_of): searched for here, one row in 2^18 is such a row.  The factor is compared bit for
bit with the oracle's."""
import numpy as np
import pytest

EPS = 1e-5
REACH = 2.0 ** -44


def open_rows(K, want, seed=0):
    """[want, K] rows with two nonzero halves each whose factor is open."""
    rng = np.random.default_rng(seed)
    found = []
    while len(found) < want:
        a = np.exp2(rng.uniform(-3, 6, 1 << 21)).astype(np.float16)
        b = np.exp2(rng.uniform(-3, 6, 1 << 21)).astype(np.float16)
        mean = (a.astype(np.float64) ** 2 + b.astype(np.float64) ** 2) / K + np.float64(np.float32(EPS))
        y = 1.0 / np.sqrt(mean)
        for i in np.nonzero((y * (1 - REACH)).astype(np.float32) != (y * (1 + REACH)).astype(np.float32))[0]:
            row = np.zeros(K, np.float16)
            row[rng.integers(K // 2)], row[K // 2 + rng.integers(K // 2)] = a[i], b[i]
            found.append(row)
    return np.stack(found[:want])


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from tests import gpu_util
    return gpu_util


@pytest.mark.gpu
@pytest.mark.parametrize("K", [64, 520, 4096, 5000, 8704, 16384])         # 1, 1, 1 or 2, 2, 2 or 6, 2 or 8 groups of eight per thread
@pytest.mark.parametrize("copies", [1, 300])                             # few rows, and more than the device has compute units
def test_open_rows(G, oracle, K, copies):
    import torch
    from paper_2509_09090_amd import binding as B
    X = np.repeat(open_rows(K, 3), copies, 0)
    X[1::7] = np.float16(0.25)                                            # ordinary rows between them
    gamma = (1 + 0.1 * np.random.default_rng(1).standard_normal(K)).astype(np.float16)
    _, y_o = oracle.rmsnorm_rows(X, gamma, EPS)
    q_o, s_o, _ = oracle.quantize_rows(y_o)
    Xq = torch.zeros((len(X), K // 2), dtype=torch.uint8, device="cuda")
    sx = torch.zeros((len(X),), dtype=torch.float16, device="cuda")
    y = torch.zeros(X.shape, dtype=torch.float16, device="cuda")
    B.sqap_rmsnorm_quantize_act(G.to_dev(X), None, G.to_dev(gamma), EPS, Xq, sx, y_out=y)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy().view(np.uint16), y_o.view(np.uint16))
    assert np.array_equal(sx.cpu().numpy().view(np.uint16), np.asarray(s_o).view(np.uint16))
    assert np.array_equal(Xq.cpu().numpy(), q_o)


@pytest.mark.gpu
def test_open_rows_in_the_step(G, oracle):
    """The first norm of a decode step, its token open: the cache row it appends is the chain of launches' to the bit."""
    import torch
    from paper_2509_09090_amd import binding as B
    from tests.test_gpu_decoder_step import _model
    hidden, H, d = 512, 4, 128
    host, dev, _, gf, head = _model(oracle, G, np.random.default_rng(3), hidden, H, d, 1408, 1, 1000, 2)
    w, kv = dev[0]
    dec = B.sqap_decoder_create([(w.qkv, w.o, w.gate_up, w.down, w.gamma_attn, w.gamma_mlp, kv)], H, d, G.to_dev(gf), head)
    pos = G.to_dev(np.array([0], np.int32))
    logits = torch.zeros((1000,), dtype=torch.float16, device="cuda")
    xq, sx = torch.zeros((1, hidden // 2), dtype=torch.uint8, device="cuda"), torch.zeros((1,), dtype=torch.float16, device="cuda")
    qkv, row = torch.zeros((1, 3 * hidden), dtype=torch.float16, device="cuda"), torch.zeros((1, 2 * hidden), dtype=torch.float16, device="cuda")
    ws = torch.zeros((max(256, B.sqap_workspace_bytes(1, 3 * hidden, hidden)),), dtype=torch.uint8, device="cuda")
    for x in open_rows(hidden, 4, seed=2):
        x = G.to_dev(x)
        dec.step(x, pos, 0, logits)
        B.sqap_rmsnorm_quantize_act(x[None], None, w.gamma_attn, EPS, xq, sx)
        B.sqap_w4a4_linear(xq, sx, w.qkv, qkv, None, ws)
        B.sqap_rope_append(qkv, pos, H, d, row)
        torch.cuda.synchronize()
        assert dec.status() == 0
        assert torch.equal(kv[:1].view(torch.int16), row.view(torch.int16))
    dec.free()
    head.free()


def test_the_search_finds_open_rows():
    rows = open_rows(256, 2)
    assert rows.shape == (2, 256) and (rows != 0).sum() == 4
