"""The work that is timed: calls a fine-tuning step makes of this library.

Every case is one training-step unit -- forward and backward together -- of a
layer that the library serves, through its public entry points:

  attn    attn_fwd + attn_bwd on token-major Q, K, V (self- and
          cross-attention, MHA and GQA, causal / key padding / no mask, bf16
          and fp32 storage), outputs and workspace kept by the caller
  proj    the three products of a linear layer (Y, dX, dW), bf16 or fp32
  lora    the six products of a LoRA adapter (H = X A, U = H B, dH, dB, dA, dX)
  block   QKV projection, attention on the packed buffer, output projection
          and their full backward through torch.autograd

Sizes are those of synth.py's workloads and of the benchmark's projection
products, with ragged ones of the same ranges between them.
"""
import math

import torch

from paper_2607_21624_amd import autograd as ag
from paper_2607_21624_amd import fbl

DEVICE = "cuda"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


# ------------------------------------------------------------------- the cases
def _attn(name, B, S, Hq, Hkv, d, dtype, mask, S_kv=0, len_lo=0):
    c = dict(kind="attn", B=B, S=S, S_kv=S_kv or S, Hq=Hq, Hkv=Hkv, d=d, dtype=dtype, mask=mask, len_lo=len_lo)
    return dict(c, name=name) if name else c


def _proj(name, M, K, N, dtype):
    c = dict(kind="proj", M=M, K=K, N=N, dtype=dtype)
    return dict(c, name=name) if name else c


def _lora(name, M, K, N, r):
    c = dict(kind="lora", M=M, K=K, N=N, r=r, dtype="bf16")
    return dict(c, name=name) if name else c


def _block(name, B, S, Hq, Hkv, d):
    c = dict(kind="block", B=B, S=S, Hq=Hq, Hkv=Hkv, d=d, dtype="bf16")
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a toy model kept in fp32 (unit tests, debugging runs); launches and latency
        _attn("attn_tiny_f32", 1, 64, 2, 2, 32, "f32", "none"),
        # an encoder batch of short padded sentences, BERT-base-like: 96 (batch, head) pairs, at most 128 keys
        _attn("attn_bert_keypad", 8, 128, 12, 12, 64, "bf16", "keypad", len_lo=32),
        # a decoder's cross-attention over padded audio frames, Whisper-large-like: both lengths ragged
        _attn("attn_whisper_cross", 4, 448, 20, 20, 64, "bf16", "keypad", S_kv=300, len_lo=100),
        # a causal decoder in fp32 at an ordinary size whose length fills no tile
        _attn("attn_f32_causal", 2, 500, 12, 12, 64, "f32", "causal"),
        # a causal decoder batch, GPT-2-medium-like
        _attn("attn_gpt2_causal", 4, 1024, 16, 16, 64, "bf16", "causal"),
        # grouped-query attention, Llama-3.2-1B-like
        _attn("attn_llama1b_gqa", 2, 2048, 32, 8, 64, "bf16", "causal"),
        # the largest: Llama-7B-like causal attention, the benchmark's default
        _attn("attn_llama7b_causal", 1, 4096, 32, 32, 128, "bf16", "causal"),
        # one linear layer, 512 tokens, the benchmark's projection shape
        _proj("proj_512_2048_8192", 512, 2048, 8192, "bf16"),
        # a fused QKV projection of hidden 768 over a packed batch whose token count fills no tile
        _proj("proj_1000_768_2304", 1000, 768, 2304, "bf16"),
        # a linear layer kept in fp32
        _proj("proj_f32_512_768_3072", 512, 768, 3072, "f32"),
        # a rank-16 adapter of a square hidden-2048 projection, 512 tokens
        _lora("lora_512_2048_r16", 512, 2048, 2048, 16),
        # a whole attention block of a GQA layer, 4096 tokens, Llama-3.2-1B-like
        _block("block_llama1b", 2, 2048, 32, 8, 64),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["attn"] * 4 + ["cross", "attn_f32", "attn_f32", "proj", "proj", "proj_f32", "lora", "block"])
    while True:
        if kind in ("attn", "cross", "attn_f32"):
            f32 = kind == "attn_f32"
            Hq = rng.choice([2, 4, 8, 12, 16] if f32 else [4, 8, 12, 16, 20, 32])
            Hkv = Hq // rng.choice([g for g in (1, 1, 1, 2, 4, 8) if Hq % g == 0])
            d = rng.choice([32, 64, 64, 128] if f32 else [32, 64, 64, 64, 128, 128, 128])
            B = _log(rng, 1, 4 if f32 else 8)
            S = _log(rng, 32, 1024 if f32 else 4096)
            S_kv = S
            mask = rng.choice(["none", "causal", "causal", "causal", "keypad"])
            if kind == "cross" or (f32 and rng.random() < 0.2):
                S, S_kv = _log(rng, 16, 1024), _log(rng, 16, 1024 if f32 else 1500)
                mask = rng.choice(["none", "keypad"])
            c = _attn("", B, S, Hq, Hkv, d, "f32" if f32 else "bf16", mask, S_kv=S_kv,
                      len_lo=max(1, S_kv // 3) if mask == "keypad" else 0)
            if 14.0 * d * B * Hq * S * S_kv <= (1.2e10 if f32 else 9.6e11) * (0.5 if mask != "causal" else 1.0):
                return c
        elif kind == "proj":
            step = rng.choice([64, 64, 8])  # contraction lengths are multiples of 8
            c = _proj("", 8 * _log(rng, 8, 1024), step * _log(rng, 512 // step, 8192 // step),
                      step * _log(rng, 512 // step, 12288 // step), "bf16")
            if 6.0 * c["M"] * c["K"] * c["N"] <= 3e11:
                return c
        elif kind == "proj_f32":
            c = _proj("", _log(rng, 32, 1024), _log(rng, 64, 3072), _log(rng, 64, 3072), "f32")
            if 6.0 * c["M"] * c["K"] * c["N"] <= 7.3e9:
                return c
        elif kind == "lora":
            return _lora("", 8 * _log(rng, 16, 512), 64 * _log(rng, 8, 64), 64 * _log(rng, 8, 64), rng.choice([8, 16, 32, 64]))
        else:
            d = rng.choice([64, 128])
            Hkv, G = rng.choice([2, 4, 8, 12]), rng.choice([1, 2, 4])
            c = _block("", _log(rng, 1, 4), 8 * _log(rng, 16, 256), Hkv * G, Hkv, d)
            hid = Hkv * G * d
            if hid <= 4096 and 6.0 * c["B"] * c["S"] * hid * (2 * hid + 2 * Hkv * d) <= 2e11:
                return c


# ------------------------------------------------------------------ the inputs
def _randn(gen, shape, dtype, scale=1.0):
    x = torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32)
    return (x * scale if scale != 1.0 else x).to(dtype)


def _inputs(case, seed):
    """The inputs alone, from the seed: activations and gradients ~ N(0, 1), weights ~ N(0, 1 / fan-in)."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    dt = DTYPES[case["dtype"]]
    if case["kind"] == "attn":
        B, S, T, Hq, Hkv, d = (case[k] for k in ("B", "S", "S_kv", "Hq", "Hkv", "d"))
        s = {"q": _randn(gen, (B, S, Hq * d), dt), "k": _randn(gen, (B, T, Hkv * d), dt),
             "v": _randn(gen, (B, T, Hkv * d), dt), "do": _randn(gen, (B, S, Hq * d), dt), "kv_len": None}
        if case["mask"] == "keypad":
            s["kv_len"] = torch.randint(case["len_lo"], T + 1, (B,), generator=gen, device=DEVICE, dtype=torch.int32)
        return s
    if case["kind"] == "proj":
        M, K, N = case["M"], case["K"], case["N"]
        return {"x": _randn(gen, (M, K), dt), "w": _randn(gen, (K, N), dt, K ** -0.5), "dy": _randn(gen, (M, N), dt)}
    if case["kind"] == "lora":
        M, K, N, r = case["M"], case["K"], case["N"], case["r"]
        return {"x": _randn(gen, (M, K), dt), "a": _randn(gen, (K, r), dt, K ** -0.5),
                "b": _randn(gen, (r, N), dt, r ** -0.5), "dy": _randn(gen, (M, N), dt)}
    B, S, Hq, Hkv, d = (case[k] for k in ("B", "S", "Hq", "Hkv", "d"))
    hid = Hq * d
    return {"x": _randn(gen, (B, S, hid), dt), "w_qkv": _randn(gen, (hid, (Hq + 2 * Hkv) * d), dt, hid ** -0.5),
            "w_o": _randn(gen, (hid, hid), dt, hid ** -0.5), "dy": _randn(gen, (B, S, hid), dt)}


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["kind"] == "attn":  # the layer's buffers, kept by a training program from step to step
        B, S, Hq, Hkv = case["B"], case["S"], case["Hq"], case["Hkv"]
        s["o"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((B, Hq, S), dtype=torch.float32, device=DEVICE)
        s["dq"], s["dk"], s["dv"] = torch.empty_like(s["q"]), torch.empty_like(s["k"]), torch.empty_like(s["v"])
        need = fbl.fbl_attn_bwd_workspace(fbl.layout_of(s["q"], Hq), fbl.layout_of(s["k"], Hkv))
        s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEVICE)
    elif case["kind"] == "proj":
        s["y"] = torch.empty_like(s["dy"])
        s["dx"], s["dw"] = torch.empty_like(s["x"]), torch.empty_like(s["w"])
    elif case["kind"] == "lora":
        s["h"] = torch.empty((case["M"], case["r"]), dtype=s["x"].dtype, device=DEVICE)
        s["dh"], s["u"], s["dx"] = torch.empty_like(s["h"]), torch.empty_like(s["dy"]), torch.empty_like(s["x"])
        s["da"], s["db"] = torch.empty_like(s["a"]), torch.empty_like(s["b"])
    else:
        for k in ("x", "w_qkv", "w_o"):
            s[k].requires_grad_(True)
    return s


# --------------------------------------------------------------------- one pass
def run(s):
    c = s["case"]
    if c["kind"] == "attn":
        causal = c["mask"] == "causal"
        fbl.attn_fwd(s["q"], s["k"], s["v"], c["Hq"], c["Hkv"], causal=causal, kv_len=s["kv_len"], out=s["o"],
                     lse=s["lse"])
        fbl.attn_bwd(s["q"], s["k"], s["v"], s["o"], s["do"], s["lse"], c["Hq"], c["Hkv"], causal=causal,
                     kv_len=s["kv_len"], dq=s["dq"], dk=s["dk"], dv=s["dv"], workspace=s["workspace"])
        return s["o"], s["lse"], s["dq"], s["dk"], s["dv"]
    if c["kind"] == "proj":
        return (fbl.proj(fbl.FBL_PROJ_FWD, s["x"], s["w"], out=s["y"]),
                fbl.proj(fbl.FBL_PROJ_BWD_DATA, s["dy"], s["w"], out=s["dx"]),
                fbl.proj(fbl.FBL_PROJ_BWD_WEIGHT, s["x"], s["dy"], out=s["dw"]))
    if c["kind"] == "lora":
        return (fbl.proj(fbl.FBL_PROJ_FWD, s["x"], s["a"], out=s["h"]),
                fbl.proj(fbl.FBL_PROJ_FWD, s["h"], s["b"], out=s["u"]),
                fbl.proj(fbl.FBL_PROJ_BWD_DATA, s["dy"], s["b"], out=s["dh"]),
                fbl.proj(fbl.FBL_PROJ_BWD_WEIGHT, s["h"], s["dy"], out=s["db"]),
                fbl.proj(fbl.FBL_PROJ_BWD_WEIGHT, s["x"], s["dh"], out=s["da"]),
                fbl.proj(fbl.FBL_PROJ_BWD_DATA, s["dh"], s["a"], out=s["dx"]))
    qkv = ag.linear(s["x"], s["w_qkv"])
    o = ag.attention_packed(qkv, c["Hq"], c["Hkv"], causal=True)
    y = ag.linear(o, s["w_o"])
    return (y.detach(),) + torch.autograd.grad(y, (s["x"], s["w_qkv"], s["w_o"]), s["dy"])


# -------------------------------------------------------- what it cannot do without
def _pairs(c):
    """Allowed (query, key) pairs of one head, summed over the batch; key padding at its mean length."""
    if c["mask"] == "causal":
        return c["B"] * c["S"] * (c["S"] + 1) / 2
    keys = (c["len_lo"] + c["S_kv"]) / 2 if c["mask"] == "keypad" else c["S_kv"]
    return c["B"] * c["S"] * keys


def work(case):
    c = case
    es = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "attn":
        q = c["B"] * c["S"] * c["Hq"] * c["d"] * es
        k = c["B"] * c["S_kv"] * c["Hkv"] * c["d"] * es
        # Q, K, V, dO read; O, LSE, dQ, dK, dV written.  14 d per pair: 4 d forward, 10 d backward
        return {"bytes": 4 * q + 4 * k + 4 * c["B"] * c["Hq"] * c["S"], "flops": 14.0 * c["d"] * c["Hq"] * _pairs(c)}
    if c["kind"] == "proj":
        M, K, N = c["M"], c["K"], c["N"]
        return {"bytes": 2 * es * (M * K + K * N + M * N), "flops": 6.0 * M * K * N}
    if c["kind"] == "lora":
        M, K, N, r = c["M"], c["K"], c["N"], c["r"]
        return {"bytes": es * (2 * M * K + 2 * M * N + 2 * r * (K + N) + 2 * M * r), "flops": 6.0 * M * r * (K + N)}
    T, hid, wide = c["B"] * c["S"], c["Hq"] * c["d"], (c["Hq"] + 2 * c["Hkv"]) * c["d"]
    # x, dy and the weights read; y, dx and the weights' gradients written
    return {"bytes": es * (4 * T * hid + 2 * hid * wide + 2 * hid * hid),
            "flops": 6.0 * T * hid * (wide + hid) + 14.0 * hid * c["B"] * c["S"] * (c["S"] + 1) / 2}


def tolerance(case):
    # bf16: inputs exact, P, dS and the results rounded to 8 bits, fp32 sums.  A block rounds
    # at every stage between.  fp32: sums in another order over up to a few thousand terms.
    if case["dtype"] == "f32":
        return {"rel": 4e-6}
    return {"rel": 2e-2 if case["kind"] == "block" else 1e-2}


# ----------------------------------------------------------------- in 64 bits
def _exact_attn(q, k, v, do, Hq, Hkv, causal, kv_len):
    """(o, lse, dq, dk, dv) in float64, one (batch, head) at a time; scale 1/sqrt(d)."""
    B, S, T, d, G = q.shape[0], q.shape[1], k.shape[1], q.shape[2] // Hq, Hq // Hkv
    scale = 1.0 / math.sqrt(d)
    o, dq, dk, dv = (torch.zeros(x.shape, dtype=torch.float64, device=x.device) for x in (q, q, k, v))
    lse = torch.zeros((B, Hq, S), dtype=torch.float64, device=q.device)
    i = torch.arange(S, device=q.device)[:, None]
    j = torch.arange(T, device=q.device)[None, :]
    for b in range(B):
        off = (j > i) if causal else torch.zeros((S, T), dtype=torch.bool, device=q.device)
        if kv_len is not None:
            off = off | (j >= kv_len[b])
        for h in range(Hq):
            hq, hk = slice(h * d, (h + 1) * d), slice(h // G * d, (h // G + 1) * d)
            qh, kh, vh, gh = q[b, :, hq].double(), k[b, :, hk].double(), v[b, :, hk].double(), do[b, :, hq].double()
            s = ((qh @ kh.T) * scale).masked_fill_(off, -math.inf)
            l = torch.logsumexp(s, dim=1)
            p = torch.exp(s - l[:, None])
            oh = p @ vh
            ds = p * (gh @ vh.T - (gh * oh).sum(1, keepdim=True)) * scale
            o[b, :, hq], lse[b, h] = oh, l
            dq[b, :, hq] = ds @ kh
            dk[b, :, hk] += ds.T @ qh
            dv[b, :, hk] += p.T @ gh
    return o, lse, dq, dk, dv


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    if c["kind"] == "attn":
        return _exact_attn(s["q"], s["k"], s["v"], s["do"], c["Hq"], c["Hkv"], c["mask"] == "causal", s["kv_len"])
    if c["kind"] == "proj":
        x, w, dy = s["x"].double(), s["w"].double(), s["dy"].double()
        return x @ w, dy @ w.T, x.T @ dy
    if c["kind"] == "lora":
        x, a, b, dy = (s[k].double() for k in ("x", "a", "b", "dy"))
        h, dh = x @ a, dy @ b.T
        return h, h @ b, dh, h.T @ dy, x.T @ dh, dh @ a.T
    B, S, Hq, Hkv, d = (c[k] for k in ("B", "S", "Hq", "Hkv", "d"))
    hid, T = Hq * d, B * S
    x, wq, wo, dy = s["x"].double().view(T, hid), s["w_qkv"].double(), s["w_o"].double(), s["dy"].double().view(T, hid)
    qkv = x @ wq
    q, k, v = (t.reshape(B, S, -1) for t in qkv.split([hid, Hkv * d, Hkv * d], dim=1))
    o, _, dq, dk, dv = _exact_attn(q, k, v, (dy @ wo.T).view(B, S, hid), Hq, Hkv, True, None)
    dqkv = torch.cat([dq, dk, dv], dim=2).view(T, -1)
    return (o.view(T, hid) @ wo).view(B, S, hid), (dqkv @ wq.T).view(B, S, hid), x.T @ dqkv, o.view(T, hid).T @ dy
