"""The prefill GEMM's block shapes and splits against the CPU oracle: every
kernel variant with every split count on a small shape, and the planner's own
choice at the sizes where they can go wrong: rows around the row tiles of 32, 64 and 128, k
ranges with fewer iterations than k groups (hidden 256), with odd remainders
over the k groups and splits (hidden 896 and 1152, FFN 688 and 4736), more rows
than columns (blocks in row order), and every weight format.  The bound is the
parity bar of all stage tests."""
import functools

import numpy as np
import pytest
import torch

from oracle import layer as O
from paper_2607_15865_amd import binding, synth
from gpu_helpers import assert_parity, bits_to_torch_f32, cache_values, log

pytestmark = pytest.mark.gpu

SHAPES = {
    "h256": synth.CONFIGS["tiny"],
    "h896": synth.replace(synth.CONFIGS["qwen05b"], ffn=4736, max_seq=512),
    "h1152": synth.LayerConfig("h1152", 1152, 9, 3, 128, 1024, 128, 1e-6, 1e4, 512, 8, 7),
}
FORMATS = {"int4": {}, "zeros": dict(with_zeros=True), "int8": dict(fmt="int8"), "bf16": dict(fmt="bf16")}
CASES = ([("h256", "int4", T) for T in (9, 32, 33, 65, 127)] +
         [("h896", f, T) for f, Ts in (("int4", (31, 64, 129, 300)), ("zeros", (33, 200)), ("int8", (65,)), ("bf16", (64, 97, 300))) for T in Ts] +
         [("h1152", f, T) for f, Ts in (("int4", (9, 96, 257)), ("zeros", (64,)), ("int8", (10, 130)), ("bf16", (33,))) for T in Ts])


@functools.lru_cache(maxsize=1)
def layer(shape, fmt):
    cfg = SHAPES[shape]
    w = synth.make_layer(cfg, 0, **FORMATS[fmt])
    return cfg, w, O.dequant_layer(w, cfg), binding.Layer(cfg, w)


@pytest.mark.parametrize("shape,fmt,T", CASES)
def test_prefill_gemm_plan(shape, fmt, T):
    cfg, w, W, lay = layer(shape, fmt)
    log(f"prefill {shape} {fmt} T={T}")
    lay.set_decode_path(1)                       # the prefill kernels for every T
    bits = synth.activations(cfg, synth.TID_X_PREFILL, T)
    x = bits_to_torch_f32(bits)
    k, v = lay.new_cache(1, 0)
    outs = []
    for _ in range(2):                           # a second call finds the first one's counters and partial sums
        y = torch.full_like(x, float("nan"))
        lay.prefill(x, torch.arange(T, dtype=torch.int32, device="cuda"), k, v, y)
        torch.cuda.synchronize()
        outs.append(y)
    assert lay.error() == 0
    assert torch.equal(outs[0], outs[1]), "the k groups and splits add in a fixed order"
    yo, ko, vo = O.prefill(w, cfg, O.bf16_to_f64(bits), np.arange(T), W=W)
    assert_parity(outs[0].cpu().numpy(), yo, "y")
    assert_parity(cache_values(k)[0][:, :T].transpose(1, 0, 2), ko, "new K")
    assert_parity(cache_values(v)[0][:, :T].transpose(1, 0, 2), vo, "new V")
    assert not np.any(cache_values(k)[0][:, T:]), "slots past the prompt are untouched"


@pytest.mark.parametrize("fmt", ["int4", "bf16"])
def test_workspace_does_not_shrink_with_longer_prompts(fmt):
    """A shape whose k splits need more for 160 rows (16-bit: 32) than for some longer
    prompts: a workspace for a longer prompt has to serve a shorter one."""
    cfg = synth.LayerConfig("wide", 1024, 8, 2, 128, 7168, 128, 1e-6, 1e4, 1024, 8, 9)
    if fmt == "bf16":
        cfg = synth.replace(cfg, hidden=2048, n_heads=16, n_kv_heads=4, ffn=5632)
    lay = binding.Layer(cfg, synth.make_layer(cfg, 0, **FORMATS[fmt]))
    for stage, hist in ((0, 0), (1, 100)):
        need = [binding.layer_workspace_size(lay.handle, stage, 1, T, hist) for T in range(1, 900)]
        assert all(a <= b for a, b in zip(need, need[1:])), [T + 1 for T in range(898) if need[T] > need[T + 1]]


def variants():
    """(format, group, row tile, waves, k groups) of the kernels that are built."""
    for fmt, group in [(f, g) for f in ("int4", "zeros") for g in (32, 64, 128)] + [("int8", 128), ("bf16", 128)]:
        for tm, wn, kg in [(tm, wn, kg) for tm in (32, 64) for wn, kg in ((4, 1), (4, 2), (2, 4))] + [(128, 4, 1)]:
            if tm == 128 and (fmt != "int4" or group == 32):
                continue
            if tm == 64 and ((fmt == "bf16" and kg > 1) or (fmt == "zeros" and group == 32 and wn == 2)):
                continue
            yield fmt, group, tm, wn, kg


@functools.lru_cache(maxsize=1)
def variant_layer(fmt, group):
    cfg = synth.replace(SHAPES["h1152"], group_size=group)        # 9 iterations of 128 k; down 8
    w = synth.make_layer(cfg, 0, **FORMATS[fmt])
    T = 300
    bits = synth.activations(cfg, synth.TID_X_PREFILL, T)
    return cfg, T, bits, O.prefill(w, cfg, O.bf16_to_f64(bits), np.arange(T), W=O.dequant_layer(w, cfg)), binding.Layer(cfg, w)


@pytest.mark.parametrize("fmt,group,tm,wn,kg", variants())
def test_every_gemm_variant_at_every_split(fmt, group, tm, wn, kg):
    """All four GEMMs (three epilogues) on one block shape, for each split count the
    planner knows (more than two iterations per k group are not needed here)."""
    cfg, T, bits, (yo, ko, vo), lay = variant_layer(fmt, group)
    lay.set_decode_path(1)
    x = bits_to_torch_f32(bits)
    for S in [s for s in (1, 2, 3, 4, 6, 8) if s == 1 or s * kg <= 8]:
        log(f"prefill {fmt} group {group}: row tile {tm}, {wn} waves, {kg} k groups, {S} splits")
        for gemm in range(4):
            assert binding.layer_set_gemm_plan(lay.handle, gemm, tm, wn, kg, S) == 0, binding.layer_last_error()
        k, v = lay.new_cache(1, 0)
        y = torch.full_like(x, float("nan"))
        lay.prefill(x, torch.arange(T, dtype=torch.int32, device="cuda"), k, v, y)
        torch.cuda.synchronize()
        assert lay.error() == 0
        assert_parity(y.cpu().numpy(), yo, "y")
        assert_parity(cache_values(k)[0][:, :T].transpose(1, 0, 2), ko, "new K")
        assert_parity(cache_values(v)[0][:, :T].transpose(1, 0, 2), vo, "new V")


def test_gemm_plan_refuses_what_is_not_built():
    lay = variant_layer("zeros", 32)[4]
    for plan in ((128, 4, 1, 1), (64, 2, 4, 1), (32, 2, 2, 1), (33, 4, 1, 1), (32, 4, 1, 0), (32, 4, 2, 5)):
        assert binding.layer_set_gemm_plan(lay.handle, 0, *plan) == binding.W4_EUNSUPPORTED, plan
    assert binding.layer_set_gemm_plan(lay.handle, 4, 32, 4, 1, 1) == binding.W4_EINVAL
