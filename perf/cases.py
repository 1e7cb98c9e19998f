"""The work a program built on this library has it do, as cases that can be timed and compared.

A case is a dict of plain values with a "kind":

  pruned_linear  observations whose visual tokens are pruned by score, then one quantized linear over the survivors
                 (top-k + surviving rows -> int4 activations with the gather fused -> W4A4 linear)
  attn_block     the attention half of a decoder layer: RMSNorm with the pending residual, q|k|v, rotary embedding, attention,
                 output projection; over a batch of sequences or into one sequence's key/value cache
  mlp            the feed-forward half: RMSNorm with the pending residual, gate|up, SwiGLU, down
  attention      causal attention of a block of queries over a longer key sequence
  decode_attn    rotation, cache append, attention and activation quantizer of one new token over a cache
  head           final norm and vocabulary head for a few tokens
  levels         the quantized linears of several layers at decode batch sizes, one grouped launch per level
  step           a whole autoregressive step of a model with key/value caches, one token at batch 1
  observe        retention scores of a batch of observations, the three-set selection rule and the surviving rows

Inputs are drawn on the GPU from the seed: activations N(0,1) with 1 % of the channels scaled by 30 (the structure the
paper's quantizer is about), weights N(0, 0.02), as in the workload definitions.
"""
import math

import torch

from paper_2509_09090_amd import binding as B

F16, F32, F64, U8, I32 = torch.float16, torch.float32, torch.float64, torch.uint8, torch.int32
DEV = "cuda"
EPS = 1e-5
BASE = 10000.0
OUTLIER_SCALE, OUTLIER_FRAC = 30.0, 0.01
WEIGHT_STD = 0.02

# hidden, heads, head size, feed-forward width: the model shapes of the workload definitions and of the tests, and one between
MODELS = ((256, 4, 64, 512), (512, 4, 128, 1408), (1024, 8, 128, 2816), (2048, 16, 128, 5504), (4096, 32, 128, 11008))


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest whole call: 64 tokens pruned to 32, one 512 x 512 linear; launches and latency
        dict(name="toy_512", kind="pruned_linear", batch=1, n_vis=64, n_text=0, keep=32, n=512, k=512, rotate=False),
        # a few observations, an uneven number of survivors, the down projection of a small model
        dict(name="ragged_down", kind="pruned_linear", batch=3, n_vis=256, n_text=20, keep=154, n=1024, k=2816, rotate=False),
        # a decoder layer's two halves for one observation: attention into its key/value cache, with the Hadamard rotation in
        # front of q/k/v, at half of the visual tokens; feed-forward at a quarter of them
        dict(name="attn_148", kind="attn_block", model=4, batch=1, seq=148, past=0, cache=True, rotate=True),
        dict(name="mlp_84", kind="mlp", m=84, hidden=4096, ffn=11008),
        # the same halves at batched prefill, the compute-bound regime: 16 observations
        dict(name="attn_16x148", kind="attn_block", model=4, batch=16, seq=148, past=0, cache=False, rotate=False),
        dict(name="mlp_2368", kind="mlp", m=2368, hidden=4096, ffn=11008),
        # a block of new tokens behind a long history
        dict(name="attention_1k_2k", kind="attention", batch=1, sq=1024, sk=2048, heads=32, d=128),
        # one new token behind a history of several observations
        dict(name="decode_attn_1500", kind="decode_attn", heads=32, d=128, past=1500),
        # the vocabulary head for a decode batch of 8
        dict(name="head_8", kind="head", m=8, hidden=4096, vocab=32000),
        # batched decode: the linears of four layers, level by level
        dict(name="levels_4x4", kind="levels", m=4, layers=4, model=4),
        # one token of the 7B-shaped model behind 148 cached positions
        dict(name="step_7b", kind="step", model=4, layers=32, vocab=32000, past=148),
        # scores, selection rule and row list for 16 observations
        dict(name="observe_16", kind="observe", batch=16, grid=16, n_text=20, heads=32, d=128, k_attn=64, keep=128, radius=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("pruned_linear", "pruned_linear", "mlp", "attn_block", "attention", "decode_attn", "head", "levels", "step",
                       "observe"))
    if kind == "pruned_linear":
        while True:
            grid = rng.choice((8, 12, 14, 16, 24))
            n_vis = grid * grid
            c = dict(kind=kind, batch=_log(rng, 1, 16), n_vis=n_vis, n_text=rng.randrange(0, 41),
                     keep=max(1, int(n_vis * rng.uniform(0.25, 1.0))), n=_log(rng, 256, 22016),
                     k=rng.choice((_log(rng, 4, 172) * 64, rng.choice(MODELS)[0], rng.choice(MODELS)[3])), rotate=rng.random() < 0.3)
            if c["batch"] * (c["keep"] + c["n_text"]) * c["n"] * c["k"] <= 2368 * 11008 * 4096:
                return c
    if kind == "mlp":
        hidden, _, _, ffn = rng.choice(MODELS)
        return dict(kind=kind, m=_log(rng, 1, 2368), hidden=hidden, ffn=ffn)
    if kind == "attn_block":
        model = rng.randrange(len(MODELS))
        if rng.random() < 0.5:
            return dict(kind=kind, model=model, batch=_log(rng, 1, 16), seq=rng.randrange(32, 149), past=0, cache=False,
                        rotate=rng.random() < 0.3)
        return dict(kind=kind, model=model, batch=1, seq=_log(rng, 1, 512), past=rng.choice((0, _log(rng, 16, 1024))), cache=True,
                    rotate=rng.random() < 0.3)
    if kind == "attention":
        sq = _log(rng, 16, 1024)
        batch = _log(rng, 1, 16) if sq <= 300 else 1
        return dict(kind=kind, batch=batch, sq=sq, sk=sq + (rng.randrange(0, 1025) if batch == 1 else 0), heads=rng.choice((4, 8, 16, 32)),
                    d=rng.choice((64, 128, 128)))
    if kind == "decode_attn":
        return dict(kind=kind, heads=rng.choice((4, 8, 16, 32)), d=rng.choice((64, 128, 128)), past=_log(rng, 1, 3000))
    if kind == "head":
        return dict(kind=kind, m=_log(rng, 1, 64), hidden=rng.choice(MODELS)[0], vocab=rng.choice((1000, 5008, 32000)))
    if kind == "levels":
        return dict(kind=kind, m=rng.randrange(1, 9), layers=rng.randrange(1, 7), model=rng.randrange(len(MODELS)))
    if kind == "step":
        return dict(kind=kind, model=rng.randrange(len(MODELS)), layers=_log(rng, 1, 16), vocab=rng.choice((1000, 5008, 32000)),
                    past=_log(rng, 8, 1200))
    grid = rng.choice((8, 12, 14, 16, 24, 32))
    n = grid * grid
    return dict(kind="observe", batch=_log(rng, 1, 16), grid=grid, n_text=rng.randrange(1, 41), heads=rng.choice((8, 16, 32)),
                d=rng.choice((64, 128)), k_attn=max(1, n // rng.choice((3, 4, 6))), keep=n // 2 + rng.randrange(0, n // 4), radius=rng.randrange(1, 4))


# ---------------------------------------------------------------- inputs (made from the seed alone)

def _gen(seed, key):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + key)
    return g


def _acts(g, m, k):
    x = torch.randn((m, k), generator=g, device=DEV)
    outliers = torch.randperm(k, generator=g, device=DEV)[: max(1, int(round(OUTLIER_FRAC * k)))]
    x[:, outliers] *= OUTLIER_SCALE
    return x.to(F16)


def _weight16(g, n, k):
    return (torch.randn((n, k), generator=g, device=DEV) * WEIGHT_STD).to(F16)


def _gain(g, k):
    return (1.0 + 0.1 * torch.randn((k,), generator=g, device=DEV)).to(F16)


def _linear_specs(hidden, ffn):
    return ((3 * hidden, hidden), (hidden, hidden), (2 * ffn, hidden), (hidden, ffn))


def _layer_inputs(seed, layer, model):
    """fp16 weights (q|k|v, o, gate|up, down) and norm gains of one layer."""
    hidden, _, _, ffn = MODELS[model]
    g = _gen(seed, 100 + layer)
    return [_weight16(g, n, k) for n, k in _linear_specs(hidden, ffn)] + [_gain(g, hidden), _gain(g, hidden)]


def _cache(seed, layer, rows, past, hidden):
    kv = torch.zeros((rows, 2 * hidden), dtype=F16, device=DEV)
    if past:
        # keys and values as a layer's projections of normalised rows leave them: std = WEIGHT_STD * sqrt(hidden)
        kv[:past] = (torch.randn((past, 2 * hidden), generator=_gen(seed, 500 + layer), device=DEV) * WEIGHT_STD * math.sqrt(hidden)).to(F16)
    return kv


def _inputs(c, seed):
    g, kind, t = _gen(seed, 1), c["kind"], {}
    if kind == "pruned_linear":
        seq = c["n_vis"] + c["n_text"]
        t["scores"] = torch.rand((c["batch"], c["n_vis"]), generator=g, device=DEV)
        t["x"] = _acts(g, c["batch"] * seq, c["k"])
        t["w"] = _weight16(g, c["n"], c["k"])
    elif kind == "mlp":
        t["x"] = _acts(g, c["m"], c["hidden"])
        t["delta"] = (0.5 * torch.randn((c["m"], c["hidden"]), generator=g, device=DEV)).to(F16)
        t["gamma"] = _gain(g, c["hidden"])
        t["w_gu"], t["w_down"] = _weight16(g, 2 * c["ffn"], c["hidden"]), _weight16(g, c["hidden"], c["ffn"])
    elif kind == "attn_block":
        m, hidden = c["batch"] * c["seq"], MODELS[c["model"]][0]
        t["x"] = _acts(g, m, hidden)
        t["pending"] = (0.5 * torch.randn((m, hidden), generator=g, device=DEV)).to(F16)
        # pruned sequences keep their original positions: increasing, with gaps
        gaps = torch.randint(1, 3, (c["batch"], c["seq"]), generator=g, device=DEV)
        t["pos"] = (c["past"] + torch.cumsum(gaps, 1) - 1).to(I32).reshape(-1)
        t["gamma"] = _gain(g, hidden)
        t["w_qkv"], t["w_o"] = _weight16(g, 3 * hidden, hidden), _weight16(g, hidden, hidden)
        if c["cache"]:
            t["kv"] = _cache(seed, 0, c["past"] + c["seq"], c["past"], hidden)
    elif kind == "attention":
        width = c["heads"] * c["d"]
        t["q"] = (1.3 * torch.randn((c["batch"] * c["sq"], width), generator=g, device=DEV)).to(F16)
        t["kv"] = (1.3 * torch.randn((c["batch"] * c["sk"], 2 * width), generator=g, device=DEV)).to(F16)
    elif kind == "decode_attn":
        width = c["heads"] * c["d"]
        t["qkv"] = (1.3 * torch.randn((3 * width,), generator=g, device=DEV)).to(F16)
        t["kv"] = (1.3 * torch.randn((c["past"] + 1, 2 * width), generator=g, device=DEV)).to(F16)
        t["kv"][c["past"]:] = 0
        t["pos"] = torch.full((1,), c["past"], dtype=I32, device=DEV)
    elif kind == "head":
        t["x"] = _acts(g, c["m"], c["hidden"])
        t["gamma"] = _gain(g, c["hidden"])
        t["w"] = _weight16(g, c["vocab"], c["hidden"])
    elif kind == "levels":
        hidden, _, _, ffn = MODELS[c["model"]]
        t["x"] = [[_acts(g, c["m"], k) for k in (hidden, hidden, hidden, ffn)] for _ in range(c["layers"])]
    elif kind == "step":
        hidden = MODELS[c["model"]][0]
        t["x"] = _acts(g, 1, hidden).reshape(-1)
        t["pos"] = torch.full((1,), c["past"], dtype=I32, device=DEV)
        t["gamma"] = _gain(g, hidden)
        t["head"] = _weight16(g, c["vocab"], hidden)
    elif kind == "observe":
        n, s = c["grid"] * c["grid"], c["grid"] * c["grid"] + c["n_text"]
        t["q"] = torch.randn((c["batch"], c["heads"], c["d"]), generator=g, device=DEV).to(F16)
        t["k"] = torch.randn((c["batch"], s, c["heads"], c["d"]), generator=g, device=DEV).to(F16)
        t["camera"] = _cameras(c, seed)
    return t


def _cameras(c, seed):
    """Pinhole cameras that see a world point on or near the token grid of 14-pixel patches."""
    g = torch.Generator().manual_seed(int(seed) * 1009 + 7)
    patch, out = 14.0, torch.zeros((c["batch"], 26), dtype=F64)
    size = c["grid"] * patch
    for b in range(c["batch"]):
        u = torch.rand(6, generator=g, dtype=F64)
        f = (0.8 + 0.8 * float(u[0])) * size
        intrinsic = torch.tensor([[f, 0, size / 2], [0, f, size / 2], [0, 0, 1]], dtype=F64)
        rot, _ = torch.linalg.qr(torch.randn((3, 3), generator=g, dtype=F64))
        shift = torch.randn(3, generator=g, dtype=F64)
        depth = 0.5 + 1.5 * float(u[1])
        seen = torch.tensor([(float(u[2]) - 0.5) * depth * size / f, (float(u[3]) - 0.5) * depth * size / f, depth], dtype=F64)
        out[b, :9] = intrinsic.reshape(-1)
        out[b, 9:21] = torch.cat([rot, shift.reshape(3, 1)], 1).reshape(-1)
        out[b, 21:24] = rot.T @ (seen - shift)
        out[b, 24:] = patch
    return out.to(DEV)


# ---------------------------------------------------------------- what a program keeps, and one pass

def _pack(w, rotate=False):
    n, k = w.shape
    wq, sw = torch.empty((n, k // 2), dtype=U8, device=DEV), torch.empty((n,), dtype=F16, device=DEV)
    B.sqap_quantize_weight(w, wq, sw, flags=B.ROTATE_HADAMARD if rotate else 0)
    return B.sqap_weight_pack(wq, sw)


def _workspace(m, *shapes):
    return torch.zeros((max(256, max(B.sqap_workspace_bytes(m, n, k) for n, k in shapes)),), dtype=U8, device=DEV)


def _quantized(m, k):
    return torch.empty((m, k // 2), dtype=U8, device=DEV), torch.empty((m,), dtype=F16, device=DEV)


def _halves(*shape):
    return torch.empty(shape, dtype=F16, device=DEV)


class State:
    pass


def prepare(case, seed):
    c, s = case, State()
    s.case = c
    s.t = t = _inputs(c, seed)
    kind = c["kind"]
    if kind == "pruned_linear":
        s.w = _pack(t.pop("w"), c["rotate"])
        s.seq, m = c["n_vis"] + c["n_text"], c["batch"] * (c["keep"] + c["n_text"])
        s.idx = torch.empty((c["batch"], c["keep"]), dtype=I32, device=DEV)
        s.rows = torch.empty((m,), dtype=I32, device=DEV)
        s.xq, s.sx = _quantized(m, c["k"])
        s.y = _halves(m, c["n"])
        s.ws = _workspace(m, (c["n"], c["k"]))
        s.flags = B.ROTATE_HADAMARD if c["rotate"] else 0
    elif kind == "mlp":
        s.gu_w, s.down_w = _pack(t.pop("w_gu")), _pack(t.pop("w_down"))
        m, hidden, ffn = c["m"], c["hidden"], c["ffn"]
        s.xq, s.sx = _quantized(m, hidden)
        s.hq, s.sh = _quantized(m, ffn)
        s.xsum, s.gu, s.out = _halves(m, hidden), _halves(m, 2 * ffn), _halves(m, hidden)
        s.ws = _workspace(m, (2 * ffn, hidden), (hidden, ffn))
    elif kind == "attn_block":
        hidden, s.heads, s.d, _ = MODELS[c["model"]]
        m = c["batch"] * c["seq"]
        s.qkv_w, s.o_w = _pack(t.pop("w_qkv"), c["rotate"]), _pack(t.pop("w_o"))
        s.flags = B.ROTATE_HADAMARD if c["rotate"] else 0
        s.xq, s.sx = _quantized(m, hidden)
        s.xsum, s.qkv, s.attn, s.out = _halves(m, hidden), _halves(m, 3 * hidden), _halves(m, hidden), _halves(m, hidden)
        s.ws = _workspace(m, (3 * hidden, hidden), (hidden, hidden))
    elif kind == "attention":
        s.o = _halves(c["batch"] * c["sq"], c["heads"] * c["d"])
    elif kind == "decode_attn":
        width = c["heads"] * c["d"]
        s.o = _halves(width)
        s.xq, s.sx = _quantized(1, width)
        s.counter = torch.zeros((1,), dtype=I32, device=DEV)
    elif kind == "head":
        s.w = _pack(t.pop("w"))
        s.xq, s.sx = _quantized(c["m"], c["hidden"])
        s.y = _halves(c["m"], c["vocab"])
        s.ws = _workspace(c["m"], (c["vocab"], c["hidden"]))
    elif kind == "levels":
        hidden, _, _, ffn = MODELS[c["model"]]
        s.groups, s.levels, s.keep = [], [], []
        for layer in range(c["layers"]):
            qkv, o, gu, down, _, _ = _layer_inputs(seed, layer, c["model"])
            parts = ((qkv[:hidden], qkv[hidden:2 * hidden], qkv[2 * hidden:]), (o,), (gu[:ffn], gu[ffn:]), (down,))
            for x, ws in zip(t["x"][layer], parts):
                xq, sx = _quantized(c["m"], x.shape[1])
                packed = [_pack(w.contiguous()) for w in ws]
                ys = [_halves(c["m"], w.N) for w in packed]
                s.groups.append((x, xq, sx, B.sqap_group_create([(xq, sx, w, y) for w, y in zip(packed, ys)])))
                s.levels.append(ys)
    elif kind == "step":
        hidden, heads, d, _ = MODELS[c["model"]]
        layers, s.kv = [], []
        for layer in range(c["layers"]):
            qkv, o, gu, down, g1, g2 = _layer_inputs(seed, layer, c["model"])
            s.kv.append(_cache(seed, layer, c["past"] + 1, c["past"], hidden))
            layers.append((_pack(qkv), _pack(o), _pack(gu), _pack(down), g1, g2, s.kv[-1]))
        s.decoder = B.sqap_decoder_create(layers, heads, d, t["gamma"], _pack(t.pop("head")), eps=EPS, rope_base=BASE)
        s.logits = _halves(c["vocab"])
    elif kind == "observe":
        n = c["grid"] * c["grid"]
        s.seq = n + c["n_text"]
        s.scores = torch.empty((c["batch"], n), dtype=F32, device=DEV)
        nbytes = B.sqap_attn_scores_workspace_bytes(c["batch"], s.seq, c["heads"], c["d"], n)
        s.ws = torch.zeros((nbytes,), dtype=U8, device=DEV) if nbytes else None
        s.cap = max(c["keep"], min(n, c["k_attn"] + (2 * c["radius"] + 1) ** 2))
        s.idx = torch.empty((c["batch"], s.cap), dtype=I32, device=DEV)
        s.count = torch.empty((c["batch"],), dtype=I32, device=DEV)
        s.rows = torch.empty((c["batch"] * (c["n_text"] + s.cap),), dtype=I32, device=DEV)
    return s


def run(s):
    c, t, kind = s.case, s.t, s.case["kind"]
    if kind == "pruned_linear":
        B.sqap_prune_rows(t["scores"], c["keep"], s.seq, 0, s.idx, s.rows)
        B.sqap_quantize_act(t["x"], s.rows, s.xq, s.sx, flags=s.flags)
        B.sqap_w4a4_linear(s.xq, s.sx, s.w, s.y, None, s.ws)
        return [s.idx, s.rows, s.xq, s.sx, s.y]
    if kind == "mlp":
        ffn = c["ffn"]
        B.sqap_rmsnorm_quantize_act(t["x"], None, t["gamma"], EPS, s.xq, s.sx, delta=t["delta"], xsum_out=s.xsum)
        B.sqap_w4a4_linear(s.xq, s.sx, s.gu_w, s.gu, None, s.ws)
        B.sqap_swiglu_quantize_act(s.gu[:, :ffn], s.gu[:, ffn:], s.hq, s.sh)
        B.sqap_w4a4_linear(s.hq, s.sh, s.down_w, s.out, None, s.ws)
        return [s.xsum, s.xq, s.sx, s.gu, s.hq, s.sh, s.out]
    if kind == "attn_block":
        h, heads, d, qkv, m = s.heads * s.d, s.heads, s.d, s.qkv, s.qkv.shape[0]
        B.sqap_rmsnorm_quantize_act(t["x"], None, t["gamma"], EPS, s.xq, s.sx, delta=t["pending"], flags=s.flags, xsum_out=s.xsum)
        B.sqap_w4a4_linear(s.xq, s.sx, s.qkv_w, qkv, None, s.ws)
        if not c["cache"]:
            B.sqap_rope(qkv[:, :2 * h], t["pos"], 2 * heads, d, BASE)      # queries and keys in one call
            key, value, kv = qkv[:, h:2 * h], qkv[:, 2 * h:], qkv
        else:
            kv = t["kv"]
            B.sqap_rope_append(qkv, t["pos"], heads, d, kv[c["past"]:], BASE)
            key, value = kv[:, :h], kv[:, h:]
        B.sqap_attention(qkv[:, :h], key, value, heads, d, s.attn, batch=c["batch"])
        B.sqap_quantize_act(s.attn, None, s.xq, s.sx)
        B.sqap_w4a4_linear(s.xq, s.sx, s.o_w, s.out, None, s.ws)
        return [s.xsum, kv, s.attn, s.out]
    if kind == "attention":
        width = c["heads"] * c["d"]
        B.sqap_attention(t["q"], t["kv"][:, :width], t["kv"][:, width:], c["heads"], c["d"], s.o, batch=c["batch"])
        return s.o
    if kind == "decode_attn":
        B.sqap_decode_attention(t["qkv"], t["pos"], c["heads"], c["d"], t["kv"], c["past"], s.o, s.xq, s.sx, s.counter)
        return [s.o, t["kv"][c["past"]], s.xq, s.sx]
    if kind == "head":
        B.sqap_rmsnorm_quantize_act(t["x"], None, t["gamma"], EPS, s.xq, s.sx)
        B.sqap_w4a4_linear(s.xq, s.sx, s.w, s.y, None, s.ws)
        return [s.xq, s.sx, s.y]
    if kind == "levels":
        for x, xq, sx, group in s.groups:
            B.sqap_quantize_act(x, None, xq, sx)
            group.run()
        return s.levels
    if kind == "step":
        s.decoder.step(t["x"], t["pos"], c["past"], s.logits)
        return [s.logits, s.kv[0][c["past"]], s.kv[-1][c["past"]]]
    B.sqap_attn_scores_batch(t["q"], t["k"], 0, c["grid"] * c["grid"], s.scores, s.ws)
    B.sqap_prune_select(s.scores, c["grid"], c["grid"], c["k_attn"], c["keep"], t["camera"], c["radius"], s.idx, s.count)
    if s.cap == c["keep"]:
        B.sqap_kept_rows(s.idx, s.seq, 0, c["grid"] * c["grid"], s.rows)
        return [s.scores, s.idx, s.count, s.rows]
    return [s.scores, s.idx, s.count]      # (sets of different sizes: a program takes the row lists one observation at a time)


# ---------------------------------------------------------------- the work that cannot be avoided

def _linear_bytes(m, n, k):
    return n * k // 2 + 2 * n + m * k // 2 + 2 * m + 2 * m * n      # packed weight, codes and scales, output


def work(case):
    c, kind = case, case["kind"]
    if kind == "pruned_linear":
        m = c["batch"] * (c["keep"] + c["n_text"])
        return {"bytes": 4 * c["batch"] * (c["n_vis"] + c["keep"]) + 4 * m + 2 * m * c["k"] + _linear_bytes(m, c["n"], c["k"]),
                "flops": 2.0 * m * c["n"] * c["k"]}
    if kind == "mlp":
        m, h, f = c["m"], c["hidden"], c["ffn"]
        return {"bytes": 6 * m * h + _linear_bytes(m, 2 * f, h) + _linear_bytes(m, h, f), "flops": 6.0 * m * h * f}
    if kind == "attn_block":
        h = MODELS[c["model"]][0]
        m, keys = c["batch"] * c["seq"], c["past"] + (c["seq"] + 1) / 2
        weights = 4 * (h * h // 2 + 2 * h)
        cache = 2 * 2 * h * (c["past"] + c["seq"]) if c["cache"] else 2 * 3 * m * h
        return {"bytes": weights + 10 * m * h + cache, "flops": 8.0 * m * h * h + 4.0 * m * keys * h}
    if kind == "attention":
        width = c["heads"] * c["d"]
        keys = c["sk"] - c["sq"] + (c["sq"] + 1) / 2
        return {"bytes": 2 * width * c["batch"] * (2 * c["sq"] + 2 * c["sk"]), "flops": 4.0 * c["batch"] * c["sq"] * keys * width}
    if kind == "decode_attn":
        width = c["heads"] * c["d"]
        return {"bytes": 2 * width * (2 * (c["past"] + 1) + 4) + width // 2, "flops": 4.0 * width * (c["past"] + 1)}
    if kind == "head":
        return {"bytes": 2 * c["m"] * c["hidden"] + _linear_bytes(c["m"], c["vocab"], c["hidden"]),
                "flops": 2.0 * c["m"] * c["vocab"] * c["hidden"]}
    if kind == "levels":
        h, _, _, f = MODELS[c["model"]]
        return {"bytes": c["layers"] * sum(_linear_bytes(c["m"], n, k) + 2 * c["m"] * k for n, k in _linear_specs(h, f)),
                "flops": 2.0 * c["layers"] * c["m"] * sum(n * k for n, k in _linear_specs(h, f))}
    if kind == "step":
        h, _, _, f = MODELS[c["model"]]
        weights = sum(n * k // 2 + 2 * n for n, k in _linear_specs(h, f))
        return {"bytes": c["layers"] * (weights + 4 * h * (c["past"] + 1) + 4 * h) + c["vocab"] * (h // 2 + 4) + 4 * h,
                "flops": c["layers"] * (2.0 * sum(n * k for n, k in _linear_specs(h, f)) + 4.0 * h * (c["past"] + 1)) + 2.0 * c["vocab"] * h}
    n, s = c["grid"] ** 2, c["grid"] ** 2 + c["n_text"]
    return {"bytes": c["batch"] * (2 * c["heads"] * c["d"] * (s + 1) + 4 * n + 208 + 4 * (2 * c["keep"] + c["n_text"])),
            "flops": 2.0 * c["batch"] * c["heads"] * c["d"] * s}


# ---------------------------------------------------------------- the results in 64 bits, and how close to them one has to be

def tolerance(case):
    kind = case["kind"]
    if kind in ("pruned_linear", "mlp", "head", "levels"):
        return "exact"                                       # defined bit for bit: integer sums, stated roundings
    if kind == "attention":
        return {"rel": 1.5e-3, "max": 1e-2}                  # 16-bit probabilities and outputs
    if kind == "decode_attn":
        return {"rel": 1.5e-3, "max": 1e-2, "differ": 0.01}  # codes of outputs that sit at a rounding edge
    if kind == "observe":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}    # 32-bit softmax; scores that tie within it
    # behind the attention, a code at a rounding edge moves by one of 15 steps
    return {"rel": 0.03, "max": 0.5}


def _quant64(v):
    """Codes (as 64-bit floats) and scale of the int4 quantizer, rows of v."""
    s = (v.abs().amax(1, keepdim=True) / 7).to(F16).to(F64).clamp(min=2.0 ** -24)
    return torch.clamp(torch.round(v / s), -8, 7), s


def _hadamard64(v):
    k = v.shape[1]
    block = k & -k
    v = v.reshape(v.shape[0], k // block, block)
    step = 1
    while step < block:
        v = v.reshape(v.shape[0], k // block, block // (2 * step), 2, step)
        v = torch.stack([v[..., 0, :] + v[..., 1, :], v[..., 0, :] - v[..., 1, :]], -2)
        step *= 2
    return v.reshape(v.shape[0], k) / math.sqrt(block)


def _pack64(codes):
    q = codes.to(torch.int64) & 15
    return (q[:, 0::2] | (q[:, 1::2] << 4)).to(U8)


def _half64(v):
    return v.to(F16).to(F64)


def _linear64(q, s, w, rotate=False):
    w = w.to(F64)
    qw, sw = _quant64(_hadamard64(w) if rotate else w)
    return (q @ qw.T) * s * sw.reshape(1, -1)


def _norm64(x, gamma):
    r = 1.0 / torch.sqrt((x * x).mean(1, keepdim=True) + EPS)
    return _half64(x * r * gamma.to(F64))


def _rope64(v, pos, heads, d):
    half = d // 2
    angle = pos.to(F64).reshape(-1, 1, 1) * BASE ** (-torch.arange(half, device=DEV, dtype=F64) * 2 / d)
    v = v.reshape(-1, heads, d)
    a, b = v[..., :half], v[..., half:]
    return _half64(torch.cat([a * angle.cos() - b * angle.sin(), b * angle.cos() + a * angle.sin()], -1)).reshape(-1, heads * d)


def _attention64(q, k, v, heads, d):
    """One sequence: the queries are its last positions."""
    sq, sk = q.shape[0], k.shape[0]
    hidden = torch.ones((sq, sk), dtype=torch.bool, device=DEV).tril(sk - sq).logical_not()
    out = []
    for h in range(heads):
        cols = slice(h * d, (h + 1) * d)
        a = (q[:, cols] @ k[:, cols].T) / math.sqrt(d)
        out.append(torch.softmax(a.masked_fill(hidden, -math.inf), 1) @ v[:, cols])
    return torch.cat(out, 1)


def _mlp64(x, gamma, w_gu, w_down):
    q, s = _quant64(_norm64(x, gamma))
    gu = _linear64(q, s, w_gu)
    g, u = _half64(gu).chunk(2, 1)
    hq, sh = _quant64(_half64(g / (1 + torch.exp(-g)) * u))
    return q, s, gu, hq, sh, _linear64(hq, sh, w_down)


def _attn64(x, pos, gamma, w_qkv, w_o, heads, d, batch, kv=None, past=0, rotate=False):
    """x: residual stream with the pending update added.  Returns (q|k|v rows after rotation or the cache, attention, o)."""
    y = _norm64(x, gamma)
    q, s = _quant64(_hadamard64(y) if rotate else y)
    query, key, value = _half64(_linear64(q, s, w_qkv, rotate)).chunk(3, 1)
    query, key = _rope64(query, pos, heads, d), _rope64(key, pos, heads, d)
    if kv is not None:
        kv = kv.to(F64)
        kv[past:] = torch.cat([key, value], 1)
        key, value = kv.chunk(2, 1)
    else:
        kv = torch.cat([query, key, value], 1)
    a = torch.cat([_attention64(*p, heads, d) for p in zip(query.chunk(batch), key.chunk(batch), value.chunk(batch))])
    return kv, a, _linear64(*_quant64(_half64(a)), w_o)


def exact(case, seed):
    c, kind = case, case["kind"]
    t = _inputs(c, seed)
    if kind == "pruned_linear":
        seq = c["n_vis"] + c["n_text"]
        idx = torch.sort(torch.sort(t["scores"], dim=1, descending=True, stable=True).indices[:, :c["keep"]], 1).values
        text = torch.arange(c["n_vis"], seq, device=DEV).expand(c["batch"], -1)
        rows = (torch.cat([idx, text], 1) + seq * torch.arange(c["batch"], device=DEV).reshape(-1, 1)).reshape(-1)
        x = t["x"][rows].to(F64)
        q, s = _quant64(_hadamard64(x) if c["rotate"] else x)
        return [idx.to(I32), rows.to(I32), _pack64(q), s.reshape(-1), _linear64(q, s, t["w"], c["rotate"])]
    if kind == "mlp":
        x = _half64(t["x"].to(F64) + t["delta"].to(F64))
        q, s, gu, hq, sh, out = _mlp64(x, t["gamma"], t["w_gu"], t["w_down"])
        return [x, _pack64(q), s.reshape(-1), gu, _pack64(hq), sh.reshape(-1), out]
    if kind == "attn_block":
        _, heads, d, _ = MODELS[c["model"]]
        x = _half64(t["x"].to(F64) + t["pending"].to(F64))
        return [x, *_attn64(x, t["pos"], t["gamma"], t["w_qkv"], t["w_o"], heads, d, c["batch"], t.get("kv"), c["past"], c["rotate"])]
    if kind == "attention":
        width = c["heads"] * c["d"]
        q, (k, v) = t["q"].to(F64), t["kv"].to(F64).split(width, 1)
        return torch.cat([_attention64(*p, c["heads"], c["d"]) for p in zip(q.chunk(c["batch"]), k.chunk(c["batch"]), v.chunk(c["batch"]))])
    if kind == "decode_attn":
        width = c["heads"] * c["d"]
        q, k, v = t["qkv"].to(F64).reshape(1, -1).split(width, 1)
        q, k = _rope64(q, t["pos"], c["heads"], c["d"]), _rope64(k, t["pos"], c["heads"], c["d"])
        kv = t["kv"].to(F64)
        kv[c["past"]] = torch.cat([k, v], 1)
        o = _attention64(q, *kv.split(width, 1), c["heads"], c["d"])
        return [o.reshape(-1), kv[c["past"]], None, _quant64(_half64(o))[1].reshape(-1)]
    if kind == "head":
        q, s = _quant64(_norm64(t["x"].to(F64), t["gamma"]))
        return [_pack64(q), s.reshape(-1), _linear64(q, s, t["w"])]
    if kind == "levels":
        hidden, _, _, ffn = MODELS[c["model"]]
        out = []
        for layer in range(c["layers"]):
            qkv, o, gu, down, _, _ = _layer_inputs(seed, layer, c["model"])
            parts = ((qkv[:hidden], qkv[hidden:2 * hidden], qkv[2 * hidden:]), (o,), (gu[:ffn], gu[ffn:]), (down,))
            for x, ws in zip(t["x"][layer], parts):
                out.append([_linear64(*_quant64(x.to(F64)), w) for w in ws])
        return out
    if kind == "step":
        # one code that falls the other way travels through every later layer: only the shallowest have a 64-bit reference
        if c["layers"] > 1:
            return None
        hidden, heads, d, _ = MODELS[c["model"]]
        x, rows = t["x"].to(F64).reshape(1, -1), []
        for layer in range(c["layers"]):
            kv = _cache(seed, layer, c["past"] + 1, c["past"], hidden)
            w_qkv, w_o, w_gu, w_down, g1, g2 = _layer_inputs(seed, layer, c["model"])
            kv, _, o = _attn64(x, t["pos"], g1, w_qkv, w_o, heads, d, 1, kv, c["past"])
            x = _half64(x + _half64(o))
            x = _half64(x + _half64(_mlp64(x, g2, w_gu, w_down)[-1]))
            rows.append(kv[c["past"]])
        return [_linear64(*_quant64(_norm64(x, t["gamma"])), t["head"]).reshape(-1), rows[0], rows[-1]]
    n = c["grid"] ** 2
    logits = torch.einsum("bhd,bshd->bhs", t["q"].to(F64), t["k"].to(F64)) / math.sqrt(c["d"])
    scores = torch.softmax(logits, 2)[:, :, :n].mean(1)
    cap = max(c["keep"], min(n, c["k_attn"] + (2 * c["radius"] + 1) ** 2))
    return [scores, None, None] + ([None] if cap == c["keep"] else [])
