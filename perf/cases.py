"""The work this library is measured on: GEMMs, feed-forward blocks, attention and whole decoder blocks
through the public binding, over the sizes, layouts, epilogues and data types they are called with.

A case is a dict of plain values; "kind" names the entry point:

  gemm       fact_gemm            one GEMM with a fused epilogue, either layout of B, bf16 or fp16
  batched    fact_gemm_batched    many equal GEMMs in one call
  large_k    fact_gemm_splitk     a small output over a very long K, with the caller's workspace
  mlp        fact_block_mlp(_f16) the two-GEMM feed-forward block (GELU or SwiGLU)
  attention  fact_attention       packed QKV in, causal or full, grouped-query or not
  block      fact_block_forward   a whole pre-norm decoder block
"""
import math

import torch

import paper_2604_26666_amd as fact

_DT = {"bf16": torch.bfloat16, "f16": torch.float16}


def listed():
    return [
        # the smallest call of the benchmark configurations: one launch that the chip is nearly idle for
        {"name": "gemm_512", "kind": "gemm", "M": 512, "N": 512, "K": 512, "nk": False, "ep": "none", "dtype": "bf16"},
        # the headline: a large training-size GEMM with bias, both operands row-major
        {"name": "gemm_8192_bias", "kind": "gemm", "M": 8192, "N": 8192, "K": 8192, "nk": False, "ep": "bias", "dtype": "bf16"},
        # a linear layer whose widths are no multiple of anything (feature counts as data gives them), row-major
        # weights: rows start at odd addresses and every edge is ragged
        {"name": "gemm_odd", "kind": "gemm", "M": 2000, "N": 1999, "K": 1777, "nk": False, "ep": "bias", "dtype": "bf16"},
        # the head of a GPT-shaped model: hidden width 768, an odd vocabulary of 50257, weights as a linear layer has them
        {"name": "lm_head_50257", "kind": "gemm", "M": 1024, "N": 50257, "K": 768, "nk": True, "ep": "none", "dtype": "bf16"},
        # the batched problem of the benchmark configurations: bound by memory traffic
        {"name": "batched_128x512", "kind": "batched", "batch": 128, "M": 512, "N": 512, "K": 512, "nk": False, "dtype": "bf16"},
        # the large-K problem: a 256 x 256 result summed over 131072 (weight gradients, Gram matrices)
        {"name": "large_k_131072", "kind": "large_k", "M": 256, "N": 256, "K": 131072, "nk": False, "dtype": "bf16"},
        # the feed-forward block of a Llama-3-8B-shaped layer in prefill, in fp16
        {"name": "mlp_swiglu_2048_f16", "kind": "mlp", "T": 2048, "d": 4096, "dff": 14336, "act": "swiglu", "res": True, "dtype": "f16"},
        # the same layer in decode: a batch of 16 sequences, one token each - the weights are read for very few rows
        {"name": "mlp_swiglu_16", "kind": "mlp", "T": 16, "d": 4096, "dff": 14336, "act": "swiglu", "res": True, "dtype": "bf16"},
        # attention of an encoder with heads of 64: every token sees every other, sequences of no round length
        {"name": "attention_full_d64", "kind": "attention", "batch": 16, "T": 500, "hq": 12, "hkv": 12, "D": 64, "causal": False},
        # causal grouped-query attention, 32 query / 8 key-value heads of 128, ragged length
        {"name": "attention_gqa_d128", "kind": "attention", "batch": 4, "T": 1999, "hq": 32, "hkv": 8, "D": 128, "causal": True},
        # whole blocks: GPT-small-shaped (LayerNorm, biases, GELU) on 8 sequences of 1024 ...
        {"name": "block_gpt_8x1024", "kind": "block", "model": "gpt", "batch": 8, "tokens": 1024},
        # ... and Llama-3-8B-shaped (RMSNorm, rotary embedding, SwiGLU) in prefill
        {"name": "block_llama_1x2048", "kind": "block", "model": "llama", "batch": 1, "tokens": 2048},
    ]


# ---- drawn cases ----------------------------------------------------------------------------

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size between lo and hi, even in its logarithm: a multiple of 64, a multiple of 8 or any number."""
    v, how = _log(rng, lo, hi), rng.random()
    step = 64 if how < 0.4 else 8 if how < 0.7 else 1
    return max(min(lo, step), v // step * step)


def draw(rng):
    """One more case: the same entry points over the ranges that the listed cases span."""
    kind = rng.choice(["gemm", "gemm", "gemm", "batched", "large_k", "mlp", "mlp", "attention", "attention", "block"])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    if kind == "gemm":
        nk, ep = rng.random() < 0.5, rng.choice(["none", "bias", "bias_gelu", "bias_res"])
        if rng.random() < 0.3:
            # every width as it comes: rows of any length, at most the listed odd case's work
            while True:
                M, N, K = _log(rng, 1, 4096), _log(rng, 16, 4096), _log(rng, 16, 4096)
                if M * N * K <= 2000 * 1999 * 1777:
                    break
        else:
            # rows of whole 16-byte pieces, as tensors of a model have them; M is any count of tokens
            M, N, K = _size(rng, 1, 8192), 8 * max(1, _size(rng, 64, 8192) // 8), 8 * max(1, _size(rng, 64, 8192) // 8)
        return {"kind": kind, "M": M, "N": N, "K": K, "nk": nk, "ep": ep, "dtype": dtype}
    if kind == "batched":
        return {"kind": kind, "batch": _log(rng, 2, 128), "M": _size(rng, 32, 512), "N": 8 * max(1, _size(rng, 32, 512) // 8),
                "K": 8 * max(1, _size(rng, 32, 1024) // 8), "nk": rng.random() < 0.5, "dtype": dtype}
    if kind == "large_k":
        return {"kind": kind, "M": 8 * max(1, _size(rng, 64, 512) // 8), "N": 8 * max(1, _size(rng, 64, 512) // 8),
                "K": 64 * max(1, _log(rng, 8192, 131072) // 64), "nk": rng.random() < 0.5, "dtype": dtype}
    if kind == "mlp":
        d, dff, act = rng.choice([(768, 3072, "gelu"), (1024, 4096, "gelu"), (2048, 5632, "swiglu"), (4096, 14336, "swiglu")])
        return {"kind": kind, "T": _size(rng, 1, 2048 if d > 2048 else 8192), "d": d, "dff": dff, "act": act,
                "res": rng.random() < 0.7, "dtype": dtype}
    if kind == "attention":
        hq, hkv, D = rng.choice([(12, 12, 64), (16, 16, 64), (32, 8, 128), (16, 4, 128)])
        T = _size(rng, 64, 4096)
        return {"kind": kind, "batch": max(1, min(_log(rng, 1, 64), 16384 // T)), "T": T, "hq": hq, "hkv": hkv, "D": D,
                "causal": rng.random() < 0.6}
    model, T = rng.choice([("gpt", 8192), ("llama", 2048)])
    tokens = _size(rng, 32, T if model == "llama" else 2048)
    return {"kind": kind, "model": model, "batch": max(1, min(_log(rng, 1, 16), T // tokens)), "tokens": tokens}


# ---- inputs -----------------------------------------------------------------------------------

class _Draw:
    """Seeded normal tensors on the GPU, drawn in fp32 and rounded once."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) * 7919 + 17)

    def __call__(self, shape, std, dtype, mean=0.0):
        x = torch.randn(shape, generator=self.g, dtype=torch.float32, device="cuda")
        return (x.mul_(std).add_(mean) if mean else x.mul_(std)).to(dtype)


_ACT = {"none": fact.ACT_NONE, "bias": fact.ACT_NONE, "bias_gelu": fact.ACT_GELU_TANH, "bias_res": fact.ACT_NONE,
        "gelu": fact.ACT_GELU_TANH, "swiglu": fact.ACT_SILU_GATE}
_MODELS = {"gpt": (768, 12, 12, 64, 3072), "llama": (4096, 32, 8, 128, 14336)}


def _ws(need):
    return torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")


def _tensors(c, seed):
    """The case's inputs alone, from the seed."""
    n, k = _Draw(seed), c["kind"]
    dt = _DT[c.get("dtype", "bf16")]
    if k in ("gemm", "batched", "large_k"):
        M, N, K, lead = c["M"], c["N"], c["K"], ((c["batch"],) if k == "batched" else ())
        # activations ~ N(0, 1); weights scaled so that results are of the size of the activations
        t = {"A": n(lead + (M, K), 1.0, dt), "B": n(lead + ((N, K) if c["nk"] else (K, N)), K ** -0.5, dt)}
        if c.get("ep", "none") != "none":
            t["bias"] = n((N,), 0.5, dt)
        if c.get("ep") == "bias_res":
            t["R"] = n((M, N), 1.0, dt)
        return t
    if k == "mlp":
        T, d, dff, gated = c["T"], c["d"], c["dff"], c["act"] == "swiglu"
        t = {"X": n((T, d), 1.0, dt), "W1": n((dff, d), 0.02, dt), "W2": n((d, dff), 0.02, dt)}
        if gated:
            t["W1u"] = n((dff, d), 0.02, dt)
        else:
            t["b1"], t["b2"] = n((dff,), 0.02, dt), n((d,), 0.02, dt)
        if c["res"]:
            t["R"] = n((T, d), 1.0, dt)
        return t
    if k == "attention":
        # a fused projection's output: query heads, key heads, value heads side by side
        return {"qkv": n((c["batch"], c["T"], (c["hq"] + 2 * c["hkv"]) * c["D"]), 1.0, dt)}
    d, hq, hkv, D, dff = _MODELS[c["model"]]
    t = {"X": n((c["batch"] * c["tokens"], d), 1.0, dt), "norm1_g": n((d,), 0.1, dt, 1.0), "norm2_g": n((d,), 0.1, dt, 1.0),
         "Wqkv": n(((hq + 2 * hkv) * D, d), 0.02, dt), "Wo": n((d, hq * D), 0.02, dt), "W1": n((dff, d), 0.02, dt), "W2": n((d, dff), 0.02, dt)}
    if c["model"] == "gpt":
        for name, size in (("norm1_b", d), ("norm2_b", d), ("bqkv", (hq + 2 * hkv) * D), ("bo", d), ("b1", dff), ("b2", d)):
            t[name] = n((size,), 0.02, dt)
    else:
        t["W1u"] = n((dff, d), 0.02, dt)
    return t


def prepare(case, seed):
    """Inputs, output buffers and the workspace the library asks for: what a program holds before the call."""
    c, k = case, case["kind"]
    s = _tensors(c, seed)
    s["case"] = c
    dt = _DT[c.get("dtype", "bf16")]
    new = lambda *shape: torch.zeros(shape, dtype=dt, device="cuda")
    f16 = int(dt == torch.float16)
    if k == "gemm":
        s["C"] = new(c["M"], c["N"])
        s["ep"] = fact.Epilogue(bias=s.get("bias"), residual=s.get("R"), ldr=c["N"], act=_ACT[c["ep"]], f16=f16)
    elif k == "batched":
        s["C"], s["ep"] = new(c["batch"], c["M"], c["N"]), fact.Epilogue(f16=f16)
    elif k == "large_k":
        s["C"], s["ep"] = new(c["M"], c["N"]), fact.Epilogue(f16=f16)
        s["need"] = fact.fact_gemm_splitk_workspace_bytes(c["M"], c["N"], c["K"], 0)
        s["ws"] = _ws(s["need"])
    elif k == "mlp":
        s["H"], s["Y"] = new(c["T"], c["dff"]), new(c["T"], c["d"])
        s["need"] = fact.fact_block_mlp_workspace_bytes(c["T"], c["d"], c["dff"], _ACT[c["act"]])
        s["ws"] = _ws(s["need"])
    elif k == "attention":
        s["O"] = new(c["batch"], c["T"], c["hq"] * c["D"])
    else:
        d, hq, hkv, D, dff = _MODELS[c["model"]]
        gpt = c["model"] == "gpt"
        s["block"] = fact.Block(c["batch"], c["tokens"], d, hq, hkv, D, dff, 0 if gpt else 1,
                                fact.ACT_GELU_TANH if gpt else fact.ACT_SILU_GATE, rope=0 if gpt else 1, eps=1e-5, rope_base=500000.0,
                                **{w: v for w, v in s.items() if w not in ("X", "case")})
        s["Y"] = new(c["batch"] * c["tokens"], d)
        s["need"] = fact.fact_block_scratch_bytes(s["block"])
        s["ws"] = _ws(s["need"])
    return s


# ---- one pass -----------------------------------------------------------------------------------

def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "gemm":
        fact.binding.check(fact.fact_gemm(c["M"], c["N"], c["K"], s["A"], c["K"], s["B"], c["K"] if c["nk"] else c["N"], c["nk"],
                                          s["C"], c["N"], s["ep"]))
        return s["C"]
    if k == "batched":
        M, N, K = c["M"], c["N"], c["K"]
        fact.binding.check(fact.fact_gemm_batched(c["batch"], M, N, K, s["A"], K, M * K, s["B"], K if c["nk"] else N, K * N, c["nk"],
                                                  s["C"], N, M * N, s["ep"]))
        return s["C"]
    if k == "large_k":
        fact.binding.check(fact.fact_gemm_splitk(c["M"], c["N"], c["K"], s["A"], c["K"], s["B"], c["K"] if c["nk"] else c["N"], c["nk"],
                                                 s["C"], c["N"], s["ep"], 0, s["ws"], s["need"]))
        return s["C"]
    if k == "mlp":
        call = fact.fact_block_mlp_f16 if c["dtype"] == "f16" else fact.fact_block_mlp
        fact.binding.check(call(c["T"], c["d"], c["dff"], s["X"], s["W1"], s.get("W1u"), s.get("b1"), _ACT[c["act"]],
                                s["W2"], s.get("b2"), s.get("R"), s["H"], s["Y"], s["ws"], s["need"]))
        return {"H": s["H"], "Y": s["Y"]}
    if k == "attention":
        B, T, hq, hkv, D = c["batch"], c["T"], c["hq"], c["hkv"], c["D"]
        w = (hq + 2 * hkv) * D
        st, base = (T * w, w, D), s["qkv"].data_ptr()
        fact.binding.check(fact.fact_attention(B, T, hq, hkv, D, base, st, base + 2 * hq * D, st, base + 2 * (hq + hkv) * D, st,
                                               s["O"], (T * hq * D, hq * D, D), int(c["causal"]), 0.0))
        return s["O"]
    fact.binding.check(fact.fact_block_forward(s["block"], s["X"], s["Y"], s["ws"], s["need"]))
    return s["Y"]


# ---- what a pass cannot do without ------------------------------------------------------------------

def _attn_flops(B, T, hq, D, causal):
    return 4.0 * B * hq * D * (T * (T + 1) / 2 if causal else T * T)


def work(case):
    c, k = case, case["kind"]
    if k in ("gemm", "batched", "large_k"):
        M, N, K, b = c["M"], c["N"], c["K"], c.get("batch", 1)
        ep = c.get("ep", "none")
        return {"bytes": 2.0 * (b * (M * K + K * N + M * N) + (N if ep != "none" else 0) + (M * N if ep == "bias_res" else 0)),
                "flops": 2.0 * b * M * N * K}
    if k == "mlp":
        T, d, dff, mats = c["T"], c["d"], c["dff"], 3 if c["act"] == "swiglu" else 2
        # H is an output of the call; the second GEMM reads it back
        return {"bytes": 2.0 * (mats * d * dff + T * d * (3 if c["res"] else 2) + 2 * T * dff), "flops": 2.0 * T * d * dff * mats}
    if k == "attention":
        B, T, hq, hkv, D = c["batch"], c["T"], c["hq"], c["hkv"], c["D"]
        return {"bytes": 2.0 * B * T * D * (2 * hq + 2 * hkv), "flops": _attn_flops(B, T, hq, D, c["causal"])}
    d, hq, hkv, D, dff = _MODELS[c["model"]]
    T, mats = c["batch"] * c["tokens"], 3 if c["model"] == "llama" else 2
    weights = d * (hq + 2 * hkv) * D + d * hq * D + mats * d * dff
    return {"bytes": 2.0 * (weights + 2 * T * d), "flops": 2.0 * T * weights + _attn_flops(c["batch"], c["tokens"], hq, D, True)}


def tolerance(case):
    """Four times the distance from 64-bit results that the arithmetic gives: one rounding to bf16 is 1.7e-3 of a
    normal result in the 2-norm and at most 2^-8 of a value, to fp16 an eighth of that; attention rounds its
    probabilities as well, the feed-forward block its hidden tensor, a whole block eight tensors on the way."""
    k, f16 = case["kind"], case.get("dtype") == "f16"
    if k in ("gemm", "batched", "large_k"):
        return {"rel": 9e-4 if f16 else 7e-3, "max": 4e-3 if f16 else 2e-2}
    if k == "mlp":
        return {"rel": 1.5e-3 if f16 else 1.2e-2, "max": 8e-3 if f16 else 5e-2}
    if k == "attention":
        return {"rel": 1e-2, "max": 8e-2}
    return {"rel": 2e-2, "max": 1e-1}


# ---- 64-bit results ---------------------------------------------------------------------------------

def _gelu(z):
    return 0.5 * z * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (z + 0.044715 * z ** 3)))


def _softmax_attention(q, k, v, causal):
    """q [B, Hq, T, D], k and v [B, Hkv, T, D], one batch entry and key/value head at a time."""
    B, hq, T, D = q.shape
    G = hq // k.shape[1]
    out = torch.empty_like(q)
    for b in range(B):
        for h in range(hq):
            s = q[b, h] @ k[b, h // G].t().contiguous() / math.sqrt(D)
            if causal:
                s.masked_fill_(torch.ones(T, T, dtype=torch.bool, device=s.device).triu_(1), -math.inf)
            out[b, h] = torch.softmax(s, dim=-1) @ v[b, h // G]
    return out


def _heads(x, B, T, H, D):
    return x.reshape(B, T, H, D).permute(0, 2, 1, 3).contiguous()


def _norm(x, g, b, rms):
    if rms:
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-5) * g
    y = x - x.mean(-1, keepdim=True)
    return y / torch.sqrt((y * y).mean(-1, keepdim=True) + 1e-5) * g + b


def _rope(x, base):
    """x [B, H, T, D], pairs (i, i + D/2)."""
    T, D = x.shape[-2:]
    ang = torch.arange(T, dtype=torch.float64, device=x.device)[:, None] * base ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device=x.device) / D)
    c, s, lo, hi = ang.cos(), ang.sin(), x[..., : D // 2], x[..., D // 2:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1)


def _mlp(x, t):
    z = x @ t["W1"].t()
    if "W1u" in t:
        h = z * torch.sigmoid(z) * (x @ t["W1u"].t())
    else:
        h = _gelu(z + t["b1"])
    y = h @ t["W2"].t()
    return h, (y + t["b2"] if "b2" in t else y)


def exact(case, seed):
    c, k = case, case["kind"]
    t = {n: v.double() for n, v in _tensors(c, seed).items()}
    if k in ("gemm", "batched", "large_k"):
        if k == "batched":
            return torch.stack([a @ (b.t().contiguous() if c["nk"] else b) for a, b in zip(t["A"], t["B"])])
        z = t["A"] @ (t["B"].t() if c["nk"] else t["B"])
        if "bias" in t:
            z += t["bias"]
        if c.get("ep") == "bias_gelu":
            z = _gelu(z)
        return z + t["R"] if "R" in t else z
    if k == "mlp":
        h, y = _mlp(t["X"], t)
        return {"H": h, "Y": y + t["R"] if "R" in t else y}
    if k == "attention":
        B, T, hq, hkv, D = c["batch"], c["T"], c["hq"], c["hkv"], c["D"]
        q, kk, v = t["qkv"].split([hq * D, hkv * D, hkv * D], dim=-1)
        o = _softmax_attention(_heads(q, B, T, hq, D), _heads(kk, B, T, hkv, D), _heads(v, B, T, hkv, D), c["causal"])
        return o.permute(0, 2, 1, 3).reshape(B, T, hq * D)
    d, hq, hkv, D, dff = _MODELS[c["model"]]
    B, T, rms = c["batch"], c["tokens"], c["model"] == "llama"
    x = t["X"]
    qkv = _norm(x, t["norm1_g"], t.get("norm1_b"), rms) @ t["Wqkv"].t()
    if "bqkv" in t:
        qkv = qkv + t["bqkv"]
    q, kk, v = qkv.split([hq * D, hkv * D, hkv * D], dim=-1)
    q, kk, v = _heads(q, B, T, hq, D), _heads(kk, B, T, hkv, D), _heads(v, B, T, hkv, D)
    if rms:
        q, kk = _rope(q, 500000.0), _rope(kk, 500000.0)
    a = _softmax_attention(q, kk, v, True).permute(0, 2, 1, 3).reshape(B * T, hq * D)
    x1 = a @ t["Wo"].t() + x
    if "bo" in t:
        x1 = x1 + t["bo"]
    return _mlp(_norm(x1, t["norm2_g"], t.get("norm2_b"), rms), t)[1] + x1
