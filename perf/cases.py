"""The calls whose speed matters to a user of this library, with their inputs, their work and their exact results.

Shapes are those of the workloads in `paper_2505_07203_amd.inputs`: the small float32 configuration, the 8B shape
(d 4096, 32 / 8 heads of 128, FFN 14336) and the 32B shape (d 5120, 40 / 8 heads of 128, FFN 27648).  Most cases are
one layer's steps through the single-kernel entry points, at the launch sizes a request gives them; three are whole
calls that return logits, on models of few layers and a small vocabulary (the per-layer shapes are the full ones).
"""
import math

import numpy as np
import torch

from paper_2505_07203_amd import binding as B
from paper_2505_07203_amd import inputs as I

SHAPES = {"tiny": I.TINY, "8b": I.LLAMA8B, "32b": I.QWEN32B}
DEV = "cuda"
VOCAB = 4096            # of the wide whole-call models


# ---------------------------------------------------------------------------------------------- the cases

def listed():
    return [
        # the small float32 configuration, one request: two layers of small launches, nothing but latency
        {"name": "tiny-f32-512", "kind": "request", "shape": "tiny", "dtype": "f32", "layers": 2, "rows": 512},
        # a short request of the mixed-length workload (median 2048 tokens), three layers at full width
        {"name": "request-1500", "kind": "request", "shape": "8b", "dtype": "bf16", "layers": 3, "rows": 1500},
        # post recommendation: a 150-token post behind a cached profile of 14 000 tokens, few-rows mode
        {"name": "post-150-behind-14000", "kind": "hit", "shape": "8b", "dtype": "bf16", "layers": 3, "rows": 150,
         "cached": 14000},
        # attention of the long request (the headline length), as the full path calls it
        {"name": "attention-32768", "kind": "attention", "shape": "8b", "dtype": "bf16", "rows": 32768},
        # attention of a request of ordinary, ragged length
        {"name": "attention-1931", "kind": "attention", "shape": "8b", "dtype": "bf16", "rows": 1931},
        # float32 attention (the path that checks the others)
        {"name": "attention-f32-3000", "kind": "attention", "shape": "8b", "dtype": "f32", "rows": 3000},
        # the MLP of one chunk of a long request
        {"name": "mlp-4096", "kind": "mlp", "shape": "8b", "dtype": "bf16", "rows": 4096},
        # the MLP of the mixed workload's shortest request
        {"name": "mlp-471", "kind": "mlp", "shape": "8b", "dtype": "bf16", "rows": 471},
        # the MLP of a chunk with FP8-dynamic linear layers
        {"name": "mlp-fp8-4096", "kind": "mlp", "shape": "8b", "dtype": "fp8", "rows": 4096},
        # ... and of a short request
        {"name": "mlp-fp8-600", "kind": "mlp", "shape": "8b", "dtype": "fp8", "rows": 600},
        # float32 MLP of a short request
        {"name": "mlp-f32-1000", "kind": "mlp", "shape": "8b", "dtype": "f32", "rows": 1000},
        # the projections around attention at the 32B shape: QKV with rotary embedding, O with the residual
        {"name": "projections-32b-3072", "kind": "projections", "shape": "32b", "dtype": "bf16", "rows": 3072},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    k = rng.randrange(10)
    if k == 0:
        return {"kind": "request", "shape": "tiny", "dtype": "f32", "layers": 2, "rows": _log(rng, 32, 1024)}
    if k == 1:
        return {"kind": "request", "shape": "8b", "dtype": "bf16", "layers": 3, "rows": _log(rng, 256, 4096)}
    if k == 2:
        return {"kind": "hit", "shape": "8b", "dtype": "bf16", "layers": 3, "rows": _log(rng, 40, 400),
                "cached": rng.randint(11000, 17000)}
    if k in (3, 4):
        return {"kind": "attention", "shape": rng.choice(["8b", "8b", "32b"]), "dtype": "bf16", "rows": _log(rng, 256, 26000)}
    if k == 5:
        return {"kind": "attention", "shape": "8b", "dtype": "f32", "rows": _log(rng, 200, 4000)}
    if k in (6, 7):
        return {"kind": "mlp", "shape": rng.choice(["8b", "8b", "32b"]), "dtype": "bf16", "rows": _log(rng, 150, 4096)}
    if k == 8:
        dtype = rng.choice(["fp8", "fp8", "f32"])
        return {"kind": "mlp", "shape": "8b", "dtype": dtype, "rows": _log(rng, 150, 4096) if dtype == "fp8" else _log(rng, 100, 1200)}
    return {"kind": "projections", "shape": rng.choice(["8b", "32b"]), "dtype": "bf16", "rows": _log(rng, 150, 8192)}


# ---------------------------------------------------------------------------------------------- inputs

def _cfg(case):
    cfg = SHAPES[case["shape"]]
    if case["kind"] in ("request", "hit"):
        cfg = cfg.replace(n_layers=case["layers"])
        if case["shape"] != "tiny":
            cfg = cfg.replace(vocab_size=VOCAB)
    return cfg.replace(dtype={"f32": I.F32, "bf16": I.BF16, "fp8": I.BF16_FP8}[case["dtype"]])


def _torch_dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


class _Draw:
    """Seeded values on the GPU: weights N(0, 0.02^2), gains 1 + N(0, 0.02^2), activations N(0, 1)."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) * 7919 + 11)
        self.dtype = dtype

    def normal(self, *shape, std=1.0, mean=0.0):
        x = torch.randn(*shape, generator=self.g, device=DEV, dtype=torch.float32)
        return (x * std + mean).to(self.dtype)

    def weight(self, *shape):
        return self.normal(*shape, std=0.02)

    def gain(self, d):
        return self.normal(d, std=0.02, mean=1.0)

    def tokens(self, n, vocab):
        return torch.randint(0, vocab, (n,), generator=self.g, device=DEV).to(torch.int32).cpu().numpy()


def _layer_weights(cfg, dr):
    d, qd, kvd, F = cfg.d_model, cfg.q_dim, cfg.kv_dim, cfg.ffn_dim
    return {I.KIND_ATTN_NORM: dr.gain(d), I.KIND_WQ: dr.weight(qd, d), I.KIND_WK: dr.weight(kvd, d),
            I.KIND_WV: dr.weight(kvd, d), I.KIND_WO: dr.weight(d, qd), I.KIND_MLP_NORM: dr.gain(d),
            I.KIND_WG: dr.weight(F, d), I.KIND_WU: dr.weight(F, d), I.KIND_WD: dr.weight(d, F)}


def _model(case, seed):
    """-> config, global tensors, layers' tensors, token ids (hit: of the cached profile and the post)"""
    cfg = _cfg(case)
    dr = _Draw(seed, _torch_dtype(case))
    glob = {I.KIND_EMBED: dr.weight(cfg.vocab_size, cfg.d_model), I.KIND_FINAL_NORM: dr.gain(cfg.d_model),
            I.KIND_LM_HEAD: dr.weight(cfg.vocab_size, cfg.d_model)}
    layers = [_layer_weights(cfg, dr) for _ in range(cfg.n_layers)]
    return cfg, glob, layers, dr.tokens(case["rows"] + case.get("cached", 0), cfg.vocab_size)


def _host(t):
    t = t.cpu()
    return t.view(torch.uint16).numpy() if t.dtype == torch.bfloat16 else t.numpy()


def _attention_inputs(case, seed):
    cfg = _cfg(case)
    dr = _Draw(seed, _torch_dtype(case))
    n, hd = case["rows"], cfg.head_dim
    # queries and keys of about the size a normalised activation gives through N(0, 0.02^2) weights
    q, k = dr.normal(n, cfg.n_q_heads, hd, std=1.3), dr.normal(n, cfg.n_kv_heads, hd, std=1.3)
    v = dr.normal(n, cfg.n_kv_heads, hd, std=1.3)
    if case["dtype"] == "bf16":       # the full path hands the queries over times the softmax scale
        q = (q.float() * B.attention_q_scale(hd)).to(torch.bfloat16)
    return q, k, v


def _mlp_inputs(case, seed):
    cfg = _cfg(case)
    dr = _Draw(seed, _torch_dtype(case))
    return (dr.normal(case["rows"], cfg.d_model), dr.gain(cfg.d_model), dr.weight(cfg.ffn_dim, cfg.d_model),
            dr.weight(cfg.ffn_dim, cfg.d_model), dr.weight(cfg.d_model, cfg.ffn_dim))


def _projection_inputs(case, seed):
    cfg = _cfg(case)
    dr = _Draw(seed, _torch_dtype(case))
    n, d = case["rows"], cfg.d_model
    return (dr.normal(n, d), dr.normal(n, cfg.q_dim), dr.gain(d), dr.weight(cfg.q_dim, d), dr.weight(cfg.kv_dim, d),
            dr.weight(cfg.kv_dim, d), dr.weight(d, cfg.q_dim))


def prepare(case, seed):
    kind = case["kind"]
    cfg = _cfg(case)
    if kind in ("request", "hit"):
        cfg, glob, layers, tokens = _model(case, seed)
        chunk = I.WORKLOADS["tiny_512" if case["shape"] == "tiny" else "llama8b_mixed16"]["chunk"]
        ctx = B.Context(cfg, len(tokens), chunk)
        for k, t in glob.items():
            ctx.po_load_tensor(k, -1, _host(t))
        for l, w in enumerate(layers):
            for k, t in w.items():
                ctx.po_load_tensor(k, l, _host(t))
        st = {"ctx": ctx, "tokens": tokens, "cand": I.label_ids(cfg)}
        if kind == "hit":             # the user's profile sits in the cache; the mode suits short suffixes
            ctx.po_set_few_rows_split(True)
            ctx.po_attach_kv_cache(case["cached"])
            ctx.po_prefill_prefix(tokens[:case["cached"]], case["cached"], st["cand"])
        return st
    if kind == "attention":
        q, k, v = _attention_inputs(case, seed)
        return {"q": q, "k": k, "v": v, "o": torch.empty_like(q), "pre": case["dtype"] == "bf16"}
    if kind == "mlp":
        x, g, wg, wu, wd = _mlp_inputs(case, seed)
        wgu = B.po_op_pack_gate_up(wg, wu)
        if case["dtype"] == "fp8":
            return {"x": x, "g": g, "wgu": B.po_op_quantize_rows(wgu), "wd": B.po_op_quantize_rows(wd), "eps": cfg.rms_eps}
        return {"x": x, "g": g, "wgu": wgu, "wd": wd, "eps": cfg.rms_eps}
    x, a, g, wq, wk, wv, wo = _projection_inputs(case, seed)
    wqkv, _ = B.po_op_pack_qkv(wq, wk, wv, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim)
    cos, sin = B.po_op_rope_table(case["rows"], cfg.head_dim, cfg.rope_theta)
    vt = torch.zeros(cfg.kv_dim, (case["rows"] + 63) // 64 * 64, dtype=x.dtype, device=DEV)
    return {"x": x, "a": a, "g": g, "wqkv": wqkv, "wo": wo, "cos": cos, "sin": sin, "vt": vt, "cfg": cfg}


# ---------------------------------------------------------------------------------------------- one pass

def run(st):
    if "ctx" in st:
        if st["ctx"].__dict__.get("_kvc") is not None:
            logits, lp, _ = st["ctx"].po_prefill_prefix(st["tokens"], 0, st["cand"])
        else:
            logits, lp = st["ctx"].po_prefill(st["tokens"], st["cand"])
        return logits, lp
    if "q" in st:
        return B.po_op_attention(st["q"], st["k"], st["v"], out=st["o"], q_prescaled=st["pre"])
    if "wd" in st:
        if isinstance(st["wd"], tuple):       # FP8-dynamic: codes and scales
            h = B.po_op_linear_fp8(*B.po_op_rmsnorm_quantize(st["x"], st["g"], st["eps"]), *st["wgu"], silu_mul=True)
            return B.po_op_linear_fp8(*B.po_op_quantize_rows(h), *st["wd"], residual=st["x"])
        h = B.po_op_gate_up_silu(B.po_op_rmsnorm(st["x"], st["g"], st["eps"]), st["wgu"])
        return B.po_op_linear(h, st["wd"], residual=st["x"])
    cfg = st["cfg"]
    y = B.po_op_rmsnorm(st["x"], st["g"], cfg.rms_eps)
    q, k, vt = B.po_op_qkv_rope(y, st["wqkv"], None, st["cos"], st["sin"], cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim,
                                vt=st["vt"], q_scale=B.attention_q_scale(cfg.head_dim))
    return q, k, vt, B.po_op_linear(st["a"], st["wo"], residual=st["x"])


# ---------------------------------------------------------------------------------------------- work

def work(case):
    cfg = _cfg(case)
    n, d, F, qd, kvd = case["rows"], cfg.d_model, cfg.ffn_dim, cfg.q_dim, cfg.kv_dim
    e = 4 if case["dtype"] == "f32" else 2
    we = 1 if case["dtype"] == "fp8" else e
    if case["kind"] == "attention":
        return {"bytes": e * n * (2 * qd + 2 * kvd), "flops": 4 * qd * n * (n + 1) / 2}
    if case["kind"] == "mlp":
        return {"bytes": 2 * e * n * d + 3 * we * d * F, "flops": 6 * n * d * F}
    if case["kind"] == "projections":
        return {"bytes": e * (n * (2 * d + 2 * qd + 2 * kvd + d) + d * (2 * qd + 2 * kvd)), "flops": 2 * n * d * (2 * qd + 2 * kvd)}
    p, L = case.get("cached", 0), cfg.n_layers
    linear = d * (2 * qd + 2 * kvd) + 3 * d * F
    # (the last layer: K and V of every row, everything else for one row)
    flops = ((L - 1) * (2 * n * linear + 4 * qd * (n * p + n * (n + 1) / 2)) + 4 * n * d * kvd + 2 * (linear - 2 * d * kvd)
             + 4 * qd * (n + p) + 2 * d * cfg.vocab_size)
    return {"bytes": e * (L * linear + d * cfg.vocab_size + n * d + L * 2 * p * kvd), "flops": flops}


def tolerance(case):
    # about four times the distance from the float64 evaluation measured for the listed and some drawn cases
    if case["dtype"] == "f32":                        # 2.6e-6, 2.4e-5
        return {"rel": 1e-5, "max": 1e-4}
    if case["kind"] in ("request", "hit"):            # 1.8e-2, 5.2e-2: three layers of bf16 roundings
        return {"rel": 7e-2, "max": 0.2}
    if case["dtype"] == "fp8":                        # 9.3e-3, 0.2: a rounding can move an E4M3 code by one step
        return {"rel": 3.5e-2, "max": 0.7}
    if case["kind"] == "attention":                   # 2.2e-3, 7e-2: late rows are averages far below the first rows
        return {"rel": 1e-2, "max": 0.25}
    return {"rel": 1.2e-2, "max": 6e-2}               # 3.2e-3, 1.5e-2


# ---------------------------------------------------------------------------------------------- exact results

def _norm64(x, g, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _linear64(a, w):
    return a @ w.double().t()


def _rope64(x, pos0, theta):
    n, _, hd = x.shape
    half = hd // 2
    inv = theta ** (-torch.arange(half, dtype=torch.float64, device=DEV) / half)
    ang = torch.arange(pos0, pos0 + n, dtype=torch.float64, device=DEV)[:, None] * inv
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat((a * c - b * s, b * c + a * s), -1)


def _attention64(q, k, v, scale):
    """causal, query i at the last positions; q [n, Hq, hd], k / v [m, Hkv, hd]"""
    n, m, group = q.shape[0], k.shape[0], q.shape[1] // k.shape[1]
    out = torch.empty_like(q)
    step = max(64, min(n, (1 << 27) // m))
    for h in range(q.shape[1]):
        kh, vh = k[:, h // group].contiguous(), v[:, h // group].contiguous()
        for r0 in range(0, n, step):
            r1 = min(n, r0 + step)
            last = m - n + r1
            s = (q[r0:r1, h] * scale) @ kh[:last].t()
            rows = torch.arange(m - n + r0, last, device=DEV)[:, None]
            s.masked_fill_(torch.arange(last, device=DEV)[None] > rows, -math.inf)
            s -= s.amax(-1, keepdim=True)
            s.exp_()
            out[r0:r1, h] = (s @ vh[:last]) / s.sum(-1, keepdim=True)
    return out


def _silu_mul64(y, wg, wu):
    g = _linear64(y, wg)
    return g * torch.sigmoid(g) * _linear64(y, wu)


def _quant64(x):
    """rows of bf16 values -> what their E4M3 codes and float32 scales stand for"""
    x = x.to(torch.bfloat16).float()
    amax = x.abs().amax(-1, keepdim=True)
    safe = torch.where(amax > 0, amax, torch.ones_like(amax))
    codes = (x * (448.0 / safe)).to(torch.float8_e4m3fn)
    return codes.double() * torch.where(amax > 0, safe / 448.0, torch.ones_like(amax)).double()


def exact(case, seed):
    kind, cfg = case["kind"], _cfg(case)
    hd, theta, eps = cfg.head_dim, cfg.rope_theta, cfg.rms_eps
    if kind == "attention":
        q, k, v = (t.double() for t in _attention_inputs(case, seed))
        scale = math.log(2.0) if case["dtype"] == "bf16" else hd ** -0.5
        return _attention64(q, k, v, scale)
    if kind == "mlp":
        x, g, wg, wu, wd = _mlp_inputs(case, seed)
        y = _norm64(x.double(), g, eps)
        if case["dtype"] == "fp8":
            y = _quant64(y)
            h = _silu_mul64(y, _quant64(wg), _quant64(wu))
            return x.double() + _quant64(h) @ _quant64(wd).t()
        return x.double() + _linear64(_silu_mul64(y, wg, wu), wd)
    if kind == "projections":
        x, a, g, wq, wk, wv, wo = _projection_inputs(case, seed)
        n = case["rows"]
        y = _norm64(x.double(), g, eps)
        q = _rope64(_linear64(y, wq).view(n, -1, hd), 0, theta).reshape(n, -1) * B.attention_q_scale(hd)
        k = _rope64(_linear64(y, wk).view(n, -1, hd), 0, theta).reshape(n, -1)
        vt = torch.zeros(cfg.kv_dim, (n + 63) // 64 * 64, dtype=torch.float64, device=DEV)
        vt[:, :n] = _linear64(y, wv).t()
        return q, k, vt, x.double() + _linear64(a.double(), wo)
    cfg, glob, layers, tokens = _model(case, seed)
    n = len(tokens)
    x = glob[I.KIND_EMBED].double()[torch.from_numpy(tokens).long().to(DEV)]
    for w in layers:
        y = _norm64(x, w[I.KIND_ATTN_NORM], eps)
        q = _rope64(_linear64(y, w[I.KIND_WQ]).view(n, -1, hd), 0, theta)
        k = _rope64(_linear64(y, w[I.KIND_WK]).view(n, -1, hd), 0, theta)
        v = _linear64(y, w[I.KIND_WV]).view(n, -1, hd)
        x = x + _linear64(_attention64(q, k, v, hd ** -0.5).reshape(n, -1), w[I.KIND_WO])
        x = x + _linear64(_silu_mul64(_norm64(x, w[I.KIND_MLP_NORM], eps), w[I.KIND_WG], w[I.KIND_WU]), w[I.KIND_WD])
    z = _linear64(_norm64(x[-1], glob[I.KIND_FINAL_NORM], eps), glob[I.KIND_LM_HEAD]).cpu().numpy()
    zc = z[I.label_ids(cfg)]
    return z, zc - zc.max() - np.log(np.exp(zc - zc.max()).sum())
