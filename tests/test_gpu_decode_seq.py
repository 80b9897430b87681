"""The kernel-sequence decode against the CPU oracle where it can go wrong:
contexts around the attention's 256-key stages and their split over blocks (a
single key, the last key of a stage, more shares than some rows have stages,
shares of several stages), masks that hide whole shares, 1 to 8 rows, k ranges
that leave waves without a tile (hidden 256) or with uneven counts (hidden 896
and 1152, FFN 688 and 4736), and every weight format.  The bound is the parity
bar of all stage tests."""
import functools

import numpy as np
import pytest
import torch

from oracle import layer as O
from paper_2607_15865_amd import binding, synth
from gpu_helpers import assert_parity, bits_to_torch_f32, cache_values, log

pytestmark = pytest.mark.gpu

SHAPES = {
    "h256": synth.replace(synth.CONFIGS["tiny"], max_seq=2304),
    "h896": synth.replace(synth.CONFIGS["qwen05b"], ffn=4736, max_seq=2304),
    "h1152": synth.LayerConfig("h1152", 1152, 9, 3, 128, 1024, 128, 1e-6, 1e4, 2304, 8, 7),
    "g32": synth.replace(synth.CONFIGS["tiny"], group_size=32, max_seq=2304),
}
FORMATS = {"int4": {}, "zeros": dict(with_zeros=True), "int8": dict(fmt="int8"), "bf16": dict(fmt="bf16")}
CASES = [
    ("h256", "int4", (0,), False), ("h256", "int4", (255, 256, 1, 2303), True), ("h256", "bf16", (511, 5, 2000), False),
    ("g32", "int4", (700, 31), False), ("g32", "zeros", (1023, 1024, 1025, 12, 300, 64, 65, 2302), True),
    ("h896", "int4", (1999,), False), ("h896", "int4", (2303, 2), False), ("h896", "int4", (511, 512, 513, 0, 2200, 255), True),
    ("h896", "zeros", (768, 900, 90), False), ("h896", "int8", (2047,), True),
    ("h1152", "int4", (1500, 1600, 800, 20, 255, 257, 2303, 900), False), ("h1152", "zeros", (2048,), True),
    ("h1152", "bf16", (256, 2111), True), ("h1152", "int8", (640, 641, 127, 128, 129), False),
]


@functools.lru_cache(maxsize=1)
def layer(shape, fmt):
    cfg = SHAPES[shape]
    w = synth.make_layer(cfg, 0, **FORMATS[fmt])
    return cfg, w, O.dequant_layer(w, cfg), binding.Layer(cfg, w)


@pytest.mark.parametrize("shape,fmt,ctx,masked", CASES)
def test_sequence_decode(shape, fmt, ctx, masked):
    cfg, w, W, lay = layer(shape, fmt)
    B, ctx = len(ctx), np.array(ctx, dtype=np.int32)
    log(f"decode {shape} {fmt} ctx={ctx} masked={masked}")
    kb, vb = synth.kv_fill(cfg, B)
    bits = synth.activations(cfg, synth.TID_X_DECODE, B)
    mask = None
    if masked:                                   # the first slots: up to all but the last key
        mask = np.zeros((B, cfg.max_seq), dtype=np.float32)
        for b in range(B):
            mask[b, :ctx[b] if b % 2 == 0 else ctx[b] // 3] = -np.inf
    x = bits_to_torch_f32(bits)
    c = torch.from_numpy(ctx).cuda()
    yo, ko, vo = O.decode(w, cfg, O.bf16_to_f64(bits), ctx, O.bf16_to_f64(kb), O.bf16_to_f64(vb), ctx, W=W, mask=mask)
    outs = {}
    for path in (1, 0):
        lay.set_decode_path(path)
        outs[path] = []
        for _ in range(2):                       # the second call finds the first one's counters
            k, v = (torch.from_numpy(t.view(np.int16).copy()).cuda() for t in (kb, vb))
            y = torch.full_like(x, float("nan"))
            lay.decode(x, c, c, int(ctx.max()), k, v, y, attn_mask=None if mask is None else torch.from_numpy(mask).cuda())
            torch.cuda.synchronize()
            assert lay.error() == 0
            assert_parity(y.cpu().numpy(), yo, f"y (path {path})")
            for got, ref, what in ((k, ko, "K"), (v, vo, "V")):
                g = cache_values(got)
                assert_parity(np.stack([g[b][:, ctx[b], :] for b in range(B)]), ref, f"new {what}")
            outs[path].append(y)
    if B <= 2 and fmt == "int4" and cfg.group_size >= 64:     # the automatic path does not depend on timing
        assert torch.equal(*outs[0])


@pytest.mark.parametrize("shape,fmt,ctx,pads", [
    ("h896", "int4", (300,), (16,)), ("h1152", "int4", (500,), (301,)),          # one row, one share
    ("h896", "int4", (511, 200), (64, 199)), ("h1152", "zeros", (2000, 1999, 700, 40), (1024, 1300, 3, 40)),
    ("h256", "bf16", (900, 1023, 255), (900, 31, 255)), ("h896", "int8", (2303,), (2048,))])
@pytest.mark.parametrize("stale", [0x7FC0, 0xFF80, 0x7F80])
def test_hidden_and_unwritten_slots_may_hold_anything(shape, fmt, ctx, pads, stale):
    """Slots hidden by the mask (the first pads[b] ones of a prompt padded on the
    left) and slots past the context hold NaN or infinities in K and V, as memory
    that was never written may."""
    cfg, w, W, lay = layer(shape, fmt)
    B, ctx = len(ctx), np.array(ctx, dtype=np.int32)
    log(f"decode {shape} {fmt} ctx={ctx} pads={pads} stale={stale:#x}")
    kb, vb = synth.kv_fill(cfg, B)
    bits = synth.activations(cfg, synth.TID_X_DECODE, B)
    mask = np.zeros((B, cfg.max_seq), dtype=np.float32)
    ks, vs = kb.copy(), vb.copy()
    for b in range(B):
        mask[b, :pads[b]] = -np.inf if b % 2 == 0 else np.finfo(np.float32).min
        for t in (ks, vs):
            t[b, :, :pads[b]] = stale
            t[b, :, ctx[b]:] = stale
    yo, ko, vo = O.decode(w, cfg, O.bf16_to_f64(bits), ctx, O.bf16_to_f64(kb), O.bf16_to_f64(vb), ctx, W=W, mask=mask)
    x, c = bits_to_torch_f32(bits), torch.from_numpy(ctx).cuda()
    for path in (1, 0):
        lay.set_decode_path(path)
        k, v = (torch.from_numpy(t.view(np.int16).copy()).cuda() for t in (ks, vs))
        y = torch.full_like(x, float("nan"))
        lay.decode(x, c, c, int(ctx.max()), k, v, y, attn_mask=torch.from_numpy(mask).cuda())
        torch.cuda.synchronize()
        assert lay.error() == 0
        assert_parity(y.cpu().numpy(), yo, f"y (path {path})")


@pytest.mark.parametrize("rows,tokens", [(1, 0), (2, 0), (0, 1), (0, 2)])
def test_captured_calls_replay(rows, tokens):
    """A decode of 1 or 2 rows over 1000 keys, or a prefill_kv of 1 or 2 tokens,
    captured once and replayed on new inputs, with eager calls between the
    replays: every replay gives the eager result (the persistent launch, which
    such calls take otherwise, hands its data over under a tag that a replay
    would repeat).  Asking for it under capture is refused."""
    cfg, w, W, lay = layer("h896", "int4")
    lay.set_decode_path(0)
    n, ctx = rows or tokens, 1000
    log(f"capture: {rows} rows, {tokens} tokens")
    ws = torch.empty(max(binding.layer_workspace_size(lay.handle, 2, n, 1, ctx), binding.layer_workspace_size(lay.handle, 1, 1, n, ctx)),
                     dtype=torch.uint8, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.zeros((n, cfg.hidden), device="cuda")
    y = torch.zeros_like(x)
    shape = (rows or 1, cfg.n_kv_heads, cfg.max_seq, cfg.head_dim)
    k, v = (torch.zeros(shape, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    c = torch.full((n,), ctx, dtype=torch.int32, device="cuda")
    pos = torch.arange(ctx, ctx + n, dtype=torch.int32, device="cuda")

    def call(out, k, v):
        if rows:
            return binding.layer_decode(lay.handle, x, c, c, ctx, None, rows, k, v, out, ws, ws.numel())
        return binding.layer_prefill_kv(lay.handle, x, pos, tokens, ctx, k, v, out, ws, ws.numel())

    binding.check(call(y, k, v))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = call(y, k, v)
        if rows:
            lay.set_decode_path(2)
            refused = call(y, k, v)
            lay.set_decode_path(0)
    binding.check(captured)
    assert not rows or refused == binding.W4_EUNSUPPORTED
    for _ in range(4):
        x.normal_(generator=gen)
        k.normal_(generator=gen)
        v.normal_(generator=gen)
        k2, v2, ref = k.clone(), v.clone(), torch.zeros_like(y)
        graph.replay()
        torch.cuda.synchronize()
        got = y.clone()
        binding.check(call(ref, k2, v2))
        torch.cuda.synchronize()
        assert_parity(got.cpu().numpy(), ref.cpu().numpy(), "y of a replay")
        assert_parity(k.float().cpu().numpy(), k2.float().cpu().numpy(), "K cache of a replay")
    assert lay.error() == 0
