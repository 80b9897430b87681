"""The work that a user of this package has it do, as cases that can be timed and compared.

A case is one call of the public binding on weights and inputs drawn from a
seed: a decode step, a prefill (with or without a history), or a whole greedy
step of a model (embedding, layers, LM head).  Shapes are the package's own
decoder-layer configurations; weights, activations and caches have the
distributions of ``synth`` but are drawn on the GPU, which is faster.

Fields of a case:
  kind    "decode", "prefill" or "model";
  shape   name of a configuration in ``synth.CONFIGS``;
  fmt     weight format: "int4", "int4z" (with zero points), "int8", "int8a", "bf16";
  group   group size of the 4-bit formats;
  B, ctx  decode: sequences and the longest context (the others are at least half as long);
  mask    decode: an additive mask that hides the first slots of every sequence;
  T, hist prefill: new tokens and cached tokens before them;
  layers, vocab   model: its size.
"""
import math

import numpy as np
import torch

from paper_2607_15865_amd import synth
from paper_2607_15865_amd import binding as w4


def listed():
    return [
        # Chat on the smallest model: one token, short context; latency of a single small call.
        dict(name="decode-05b", kind="decode", shape="qwen05b", fmt="int4", group=128, B=1, ctx=512, mask=False),
        # The headline decode step: one token of the 8B-shaped layer.
        dict(name="decode-8b", kind="decode", shape="llama8b", fmt="int4", group=128, B=1, ctx=2048, mask=False),
        # Serving: a full batch of long, ragged contexts.
        dict(name="decode-7b-batch8", kind="decode", shape="qwen7b", fmt="int4", group=128, B=8, ctx=8192, mask=False),
        # Serving a checkpoint with zero points, prompts padded on the left and masked.
        dict(name="decode-8b-zeros-batch4", kind="decode", shape="llama8b", fmt="int4z", group=128, B=4, ctx=1500, mask=True),
        # One token of a layer kept in 8 bits.
        dict(name="decode-8b-int8", kind="decode", shape="llama8b", fmt="int8", group=128, B=1, ctx=4000, mask=False),
        # Speculative decoding: five draft tokens checked in one call.
        dict(name="verify-8b", kind="prefill", shape="llama8b", fmt="int4", group=128, T=5, hist=2048),
        # A short follow-up message to the smallest model.
        dict(name="prefill_kv-05b", kind="prefill", shape="qwen05b", fmt="int4", group=128, T=61, hist=250),
        # The headline prefill: a prompt of 512 tokens.
        dict(name="prefill-8b", kind="prefill", shape="llama8b", fmt="int4", group=128, T=512, hist=0),
        # The headline chunk after a history.
        dict(name="prefill_kv-8b", kind="prefill", shape="llama8b", fmt="int4", group=128, T=128, hist=1024),
        # A prompt of odd length on unquantised weights.
        dict(name="prefill-8b-bf16", kind="prefill", shape="llama8b", fmt="bf16", group=128, T=200, hist=0),
        # A long prompt, the largest call.
        dict(name="prefill-7b", kind="prefill", shape="qwen7b", fmt="int4", group=128, T=2011, hist=0),
        # A whole greedy step of a small model for four sequences: embedding, layers, logits and picks.
        dict(name="model-05b-batch4", kind="model", shape="qwen05b", fmt="int4", group=128, layers=12, vocab=152064, B=4, ctx=300),
    ]


def draw(rng):
    """One more case: shape, weight format, group size, batch, context and lengths over their whole ranges."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    shape = rng.choice(["qwen05b", "llama8b", "llama8b", "qwen7b"])
    fmt = rng.choice(["int4"] * 5 + ["int4z"] * 2 + ["int8", "int8a", "bf16"])
    group = rng.choice([128, 128, 128, 64, 32]) if fmt.startswith("int4") else 128
    c = dict(shape=shape, fmt=fmt, group=group)
    what = rng.random()
    if what < 0.45:
        return dict(kind="decode", B=rng.randint(1, 8), ctx=log_int(16, 8192), mask=rng.random() < 0.25, **c)
    if what < 0.93:
        # the longest prompts only where the listed long prompt is no smaller
        top = 2000 if fmt == "int4" and group == 128 else 800
        T = log_int(2, top)
        hist = 0 if rng.random() < 0.4 else log_int(16, 4096)
        return dict(kind="prefill", T=T, hist=hist, **c)
    c.update(shape="qwen05b", fmt="int4", group=128)
    return dict(kind="model", layers=rng.randint(2, 8), vocab=64 * log_int(500, 2376), B=rng.randint(1, 8), ctx=log_int(16, 1000), **c)


# ---------------------------------------------------------------- inputs

def config(case):
    """The case's layer configuration, with cache slots for at least its longest sequence."""
    cfg = synth.CONFIGS[case["shape"]]
    need = case["hist"] + case["T"] if case["kind"] == "prefill" else case["ctx"] + 1
    return synth.replace(cfg, group_size=case["group"], max_seq=max(cfg.max_seq, -(-need // 256) * 256))


def generator(seed, part):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1009 + part) % (1 << 62))


def host(t):
    return t.cpu().numpy()


def bf16_bits(t):
    return t.to(torch.bfloat16).view(torch.int16)


def linear(g, K, N, fmt, group):
    """One linear on the GPU, with the distributions of synth.make_linear."""
    rand = dict(generator=g, device="cuda")
    if fmt == "bf16":
        return dict(w16=bf16_bits(torch.randn((K, N), **rand) * 0.01))
    if fmt in ("int8", "int8a"):
        d = dict(scales=(torch.randn(N, **rand).abs() * (0.02 / 128)).half())
        d["q8"] = torch.randint(-128, 128, (K, N), dtype=torch.int8, **rand)
        if fmt == "int8a":
            d["zeros"] = torch.randint(96, 161, (N,), dtype=torch.uint8, **rand)
        return d
    ng = -(-K // group)
    d = dict(qweight=torch.randint(-(1 << 31), 1 << 31, (K // 8, N), dtype=torch.int64, **rand).to(torch.int32),
             scales=(torch.randn((ng, N), **rand).abs() * (0.02 / 8)).half())
    if fmt == "int4z":
        d["zeros"] = torch.randint(0, 16, (ng, N), dtype=torch.uint8, **rand)
    return d


def norm_weight(g, n):
    return bf16_bits(torch.rand(n, generator=g, device="cuda") + 0.5)


def layer_weights(cfg, fmt, seed, index=0):
    g = generator(seed, 100 + index)
    w = {name: linear(g, *cfg.linear_shape(name), fmt, cfg.group_size) for name in synth.LINEARS}
    w["attn_norm"], w["mlp_norm"] = norm_weight(g, cfg.hidden), norm_weight(g, cfg.hidden)
    return w


def to_host(w, fmt):
    """The binding's host format of layer_weights()."""
    out = {}
    for name, v in w.items():
        if isinstance(v, dict):
            lin = {k: host(t) for k, t in v.items()}
            if fmt in ("int8", "int8a", "bf16"):
                lin["format"] = "bf16" if fmt == "bf16" else "int8"
            if fmt == "int8a":
                lin["q8"] = lin["q8"].view(np.uint8)
            out[name] = lin
        else:
            out[name] = host(v).view(np.uint16)
    return out


def lm_weights(cfg, vocab, seed):
    g = generator(seed, 90)
    embed = bf16_bits(torch.randn((vocab, cfg.hidden), generator=g, device="cuda"))
    return embed, norm_weight(g, cfg.hidden), linear(g, cfg.hidden, vocab, "int4", cfg.group_size)


def hidden_states(cfg, rows, seed):
    return torch.randn((rows, cfg.hidden), generator=generator(seed, 1), device="cuda").to(torch.bfloat16).float()


def caches(cfg, batch, filled, seed, index=0):
    """K and V caches (bf16 bit patterns) with N(0, 1) values in the first `filled` slots and zeros after them."""
    g = generator(seed, 50 + index)
    out = []
    for _ in range(2):
        c = torch.zeros((batch, cfg.n_kv_heads, cfg.max_seq, cfg.head_dim), dtype=torch.int16, device="cuda")
        c[:, :, :filled] = bf16_bits(torch.randn((batch, cfg.n_kv_heads, filled, cfg.head_dim), generator=g, device="cuda"))
        out.append(c)
    return out


def contexts(case, seed):
    """Context lengths of the sequences: the longest is case["ctx"]."""
    B, ctx = case["B"], case["ctx"]
    c = torch.randint(ctx // 2, ctx + 1, (B,), generator=generator(seed, 2), device="cuda", dtype=torch.int32)
    c[B // 2] = ctx
    return c


def attention_mask(case, seed):
    """Additive mask that hides the first (at most a quarter of the) slots of every sequence."""
    B, ctx = case["B"], case["ctx"]
    pad = torch.randint(0, ctx // 4 + 1, (B, 1), generator=generator(seed, 3), device="cuda")
    slot = torch.arange(config(case).max_seq, device="cuda")[None, :]
    return torch.where(slot < pad, -math.inf, 0.0).float().contiguous()


def prepare(case, seed):
    cfg = config(case)
    s = dict(case=case)
    if case["kind"] == "model":
        B = case["B"]
        s["layers"] = [w4.Layer(cfg, to_host(layer_weights(cfg, case["fmt"], seed, i), case["fmt"])) for i in range(case["layers"])]
        embed, final_norm, head = lm_weights(cfg, case["vocab"], seed)
        s["lm"] = w4.LM(cfg, dict(vocab=case["vocab"], embed=host(embed).view(np.uint16), final_norm=host(final_norm).view(np.uint16),
                                  head={k: host(t) for k, t in head.items()}))
        s["handles"] = [l.handle for l in s["layers"]]
        kv = [caches(cfg, B, case["ctx"], seed, i) for i in range(case["layers"])]
        s["k"], s["v"] = [c[0] for c in kv], [c[1] for c in kv]
        s["ctx_lens"] = contexts(case, seed)
        s["tokens"] = torch.randint(0, case["vocab"], (B,), generator=generator(seed, 4), device="cuda", dtype=torch.int32)
        s["logits"] = torch.zeros((B, case["vocab"]), device="cuda")
        s["picks"] = torch.zeros(B, dtype=torch.int32, device="cuda")
        n = w4.model_decode_workspace_size(s["handles"], s["lm"].handle, B, case["ctx"])
        s["ws"] = torch.zeros(n, dtype=torch.uint8, device="cuda")
        return s
    s["layer"] = w4.Layer(cfg, to_host(layer_weights(cfg, case["fmt"], seed), case["fmt"]))
    if case["kind"] == "decode":
        s["x"] = hidden_states(cfg, case["B"], seed)
        s["ctx_lens"] = contexts(case, seed)
        s["k"], s["v"] = caches(cfg, case["B"], case["ctx"], seed)
        s["mask"] = attention_mask(case, seed) if case["mask"] else None
    else:
        s["x"] = hidden_states(cfg, case["T"], seed)
        s["pos"] = torch.arange(case["hist"], case["hist"] + case["T"], device="cuda", dtype=torch.int32)
        s["k"], s["v"] = caches(cfg, 1, case["hist"], seed)
    s["y"] = torch.zeros_like(s["x"])
    return s


def run(s):
    """One call; returns its output and the caches it has written its keys and values into.  (A model's
    picks are the argmax of the logits returned; between near-equal logits they fall either way.)"""
    case = s["case"]
    if case["kind"] == "decode":
        s["layer"].decode(s["x"], s["ctx_lens"], s["ctx_lens"], case["ctx"], s["k"], s["v"], s["y"], attn_mask=s["mask"])
    elif case["kind"] == "prefill":
        if case["hist"]:
            s["layer"].prefill_kv(s["x"], s["pos"], case["hist"], s["k"], s["v"], s["y"])
        else:
            s["layer"].prefill(s["x"], s["pos"], s["k"], s["v"], s["y"])
    else:
        w4.check(w4.model_decode_greedy(s["handles"], s["lm"].handle, s["tokens"], s["ctx_lens"], s["ctx_lens"], case["ctx"], case["B"],
                                        s["k"], s["v"], s["logits"], s["picks"], s["ws"], s["ws"].numel()))
        return dict(logits=s["logits"], k=s["k"][-1].view(torch.bfloat16), v=s["v"][-1].view(torch.bfloat16))
    return dict(y=s["y"], k=s["k"].view(torch.bfloat16), v=s["v"].view(torch.bfloat16))


# ---------------------------------------------------------------- what a pass cannot do without

def weight_work(cfg, fmt):
    """(bytes, multiplications per row) of a layer's weights."""
    nbytes, mults = 4 * cfg.hidden, 0
    for name in synth.LINEARS:
        K, N = cfg.linear_shape(name)
        mults += K * N
        if fmt.startswith("int4"):
            ng = -(-K // cfg.group_size)
            nbytes += K * N // 2 + ng * N * (3 if fmt == "int4z" else 2)
        else:
            nbytes += K * N * (2 if fmt == "bf16" else 1) + (0 if fmt == "bf16" else N * (3 if fmt == "int8a" else 2))
    return nbytes, mults


def layer_work(cfg, fmt, rows, sequences, keys):
    """rows new tokens over `sequences` caches; keys: (cached keys read, query-key pairs)."""
    wb, mults = weight_work(cfg, fmt)
    per_key = 4 * cfg.n_kv_heads * cfg.head_dim                 # K and V, bf16
    read, pairs = keys
    return (wb + per_key * (read + rows) + 8 * rows * cfg.hidden,
            2 * rows * mults + 4 * cfg.head_dim * cfg.n_heads * pairs)


def work(case):
    cfg = config(case)
    if case["kind"] == "prefill":
        T, L = case["T"], case["hist"]
        nbytes, flops = layer_work(cfg, case["fmt"], T, 1, (L, T * L + T * (T + 1) // 2))
        return {"bytes": nbytes, "flops": flops}
    B, keys = case["B"], case["ctx"] + (case["B"] - 1) * 3 * case["ctx"] // 4     # contexts average 3/4 of the longest
    nbytes, flops = layer_work(cfg, case["fmt"], B, B, (keys, keys + B))
    if case.get("mask"):
        nbytes += 4 * keys
    if case["kind"] == "model":
        H, V = cfg.hidden, case["vocab"]
        nbytes = nbytes * case["layers"] + H * V // 2 + 2 * V * (-(-H // cfg.group_size)) + 4 * V * B + 2 * H * B
        flops = flops * case["layers"] + 2 * B * H * V
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # The block rounds its intermediate activations to bf16, so sums in another
    # order flip single roundings of 2^-9.  Measured on the two decode paths,
    # and on a prompt cut in two, against the whole call: a layer's y moves by
    # up to 4e-4 (largest difference 3e-3), single cache entries by one bf16
    # step (5.5e-3); a 24-layer model's logits move by 1.7e-3 (1.4e-2) between
    # two runs of the same call.  About four times that:
    if case["kind"] == "model":
        return {"rel": 7e-3, "max": 0.06}
    return {"rel": 1.6e-3, "max": 0.022}


# ---------------------------------------------------------------- the same in 64 bits

def value(bits):
    return bits.view(torch.bfloat16).double()


def dequant(lin, fmt, group):
    if fmt == "bf16":
        return value(lin["w16"])
    if fmt == "int8":
        return lin["scales"].double()[None, :] * lin["q8"].double()
    if fmt == "int8a":
        return lin["scales"].double()[None, :] * (lin["q8"].view(torch.uint8).double() - lin["zeros"].double()[None, :])
    q = lin["qweight"]
    K, N = q.shape[0] * 8, q.shape[1]
    codes = torch.stack([(q >> (4 * j)) & 15 for j in range(8)], dim=1).reshape(K, N)
    g = torch.arange(K, device=q.device) // group
    z = lin["zeros"].double()[g] if "zeros" in lin else 8.0
    return lin["scales"].double()[g] * (codes.double() - z)


def rmsnorm(x, gamma, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * value(gamma)


def rope(x, pos, cfg):
    """x [rows][heads][d], the rotate-half pairing."""
    d = cfg.head_dim
    theta = float(cfg.rope_base) ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    ang = pos.double()[:, None, None] * theta
    c, s = torch.cos(ang), torch.sin(ang)
    a, b = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def attend(q, k, v, first, bias=None):
    """q [rows][heads][d] over k, v [kv heads][slots][d]; row t sees slots up to first + t."""
    rows, nq, d = q.shape
    r = nq // k.shape[0]
    n = first + rows
    hidden = torch.arange(n, device=q.device)[None, :] > first + torch.arange(rows, device=q.device)[:, None]
    out = torch.empty_like(q)
    for h in range(nq):
        s = q[:, h] @ k[h // r, :n].T / math.sqrt(d)
        if bias is not None:
            s = s + bias[:n].double()
        out[:, h] = torch.softmax(s.masked_fill(hidden, -math.inf), dim=-1) @ v[h // r, :n]
    return out


def layer_exact(case, cfg, w, x, pos, kc, vc, starts, mask=None):
    """The layer on x [rows][hidden].  starts: None for a prefill of one sequence (its first slot is
    case["hist"]), else the slot of each row's sequence.  kc, vc (64 bits) take the new keys and values."""
    W = lambda name: dequant(w[name], case["fmt"], cfg.group_size)  # noqa: E731
    rows, d = x.shape[0], cfg.head_dim
    xn = rmsnorm(x, w["attn_norm"], cfg.rms_eps)
    q = rope((xn @ W("q")).reshape(rows, cfg.n_heads, d), pos, cfg)
    k = rope((xn @ W("k")).reshape(rows, cfg.n_kv_heads, d), pos, cfg)
    v = (xn @ W("v")).reshape(rows, cfg.n_kv_heads, d)
    if starts is None:
        L = case["hist"]
        kc[0, :, L:L + rows], vc[0, :, L:L + rows] = k.transpose(0, 1), v.transpose(0, 1)
        a = attend(q, kc[0], vc[0], L)
    else:
        a = torch.empty_like(q)
        for b, at in enumerate(starts):
            kc[b, :, at], vc[b, :, at] = k[b], v[b]
            a[b:b + 1] = attend(q[b:b + 1], kc[b], vc[b], at, None if mask is None else mask[b])
    h = x + a.reshape(rows, -1) @ W("o")
    hn = rmsnorm(h, w["mlp_norm"], cfg.rms_eps)
    gate = hn @ W("gate")
    return h + (gate * torch.sigmoid(gate) * (hn @ W("up"))) @ W("down")


def exact(case, seed):
    cfg = config(case)
    if case["kind"] == "model":
        embed, final_norm, head = lm_weights(cfg, case["vocab"], seed)
        tokens = torch.randint(0, case["vocab"], (case["B"],), generator=generator(seed, 4), device="cuda", dtype=torch.int32)
        ctx = contexts(case, seed)
        x = value(embed[tokens.long()])
        for i in range(case["layers"]):
            k, v = (value(c) for c in caches(cfg, case["B"], case["ctx"], seed, i))
            x = layer_exact(case, cfg, layer_weights(cfg, case["fmt"], seed, i), x, ctx, k, v, ctx.tolist())
        logits = rmsnorm(x, final_norm, cfg.rms_eps) @ dequant(head, "int4", cfg.group_size)
        return dict(logits=logits, k=k, v=v)
    w = layer_weights(cfg, case["fmt"], seed)
    if case["kind"] == "decode":
        ctx = contexts(case, seed)
        k, v = (value(c) for c in caches(cfg, case["B"], case["ctx"], seed))
        y = layer_exact(case, cfg, w, hidden_states(cfg, case["B"], seed).double(), ctx, k, v, ctx.tolist(),
                        attention_mask(case, seed) if case["mask"] else None)
    else:
        pos = torch.arange(case["hist"], case["hist"] + case["T"], device="cuda")
        k, v = (value(c) for c in caches(cfg, 1, case["hist"], seed))
        y = layer_exact(case, cfg, w, hidden_states(cfg, case["T"], seed).double(), pos, k, v, None)
    return dict(y=y, k=k, v=v)
