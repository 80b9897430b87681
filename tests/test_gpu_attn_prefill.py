"""The prefill attention against the CPU oracle through whole layers, where its
tiling can go wrong: query tiles and 64-key stages with remainders, key ranges
of one chunk, of several, and of more chunks than the merge reads at once, for
blocks of 1, 2, 3, 4, 7 and 8 heads (registers or LDS staging) and both head
sizes.  The bound is the parity bar of all stage tests."""
import functools

import numpy as np
import pytest
import torch

from oracle import layer as O
from paper_2607_15865_amd import binding, synth
from gpu_helpers import assert_parity, bits_to_torch_f32, cache_values, log, to_cache_bits

pytestmark = pytest.mark.gpu


def shape(heads, kv, d):
    return synth.LayerConfig(f"a{heads}_{kv}_{d}", 256, heads, kv, d, 256, 64, 1e-6, 1e4, 2560, 2, 3)


CASES = [((8, 2, 128), 33, 0), ((8, 2, 128), 130, 1), ((8, 2, 128), 9, 2400), ((8, 2, 128), 500, 300), ((4, 1, 128), 64, 63),
         ((7, 1, 128), 65, 700), ((7, 1, 128), 31, 2500), ((8, 1, 128), 40, 200), ((1, 1, 128), 70, 130), ((2, 1, 128), 33, 600),
         ((6, 2, 128), 100, 64), ((14, 2, 64), 61, 250), ((14, 2, 64), 20, 2400), ((4, 1, 64), 129, 0), ((2, 2, 64), 65, 100)]


@functools.lru_cache(maxsize=1)
def layer(dims):
    cfg = shape(*dims)
    w = synth.make_layer(cfg)
    return cfg, w, O.dequant_layer(w, cfg), binding.Layer(cfg, w)


@pytest.mark.parametrize("dims,T,L", CASES)
def test_prefill_attention(dims, T, L):
    cfg, w, W, lay = layer(dims)
    log(f"prefill attention {dims} T={T} L={L}")
    lay.set_decode_path(1)                       # the prefill kernels for every T
    bits = synth.activations(cfg, synth.TID_X_PREFILL_KV, T)
    rng = np.random.default_rng(T * 10007 + L)
    kv = [to_cache_bits(O.round_bf16(rng.standard_normal((cfg.n_kv_heads, cfg.max_seq, cfg.head_dim)))) for _ in range(2)]
    k, v = (torch.from_numpy(t[None].copy()).cuda() for t in kv)
    x = bits_to_torch_f32(bits)
    pos = torch.arange(L, L + T, dtype=torch.int32, device="cuda")
    y = torch.full_like(x, float("nan"))
    if L:
        lay.prefill_kv(x, pos, L, k, v, y)
    else:
        lay.prefill(x, pos, k, v, y)
    torch.cuda.synchronize()
    assert lay.error() == 0
    kc, vc = (O.bf16_to_f64(t.view(np.uint16)) for t in kv)
    if L:
        yo, ko, vo = O.prefill_kv(w, cfg, O.bf16_to_f64(bits), np.arange(L, L + T), kc, vc, L, W=W)
    else:
        yo, ko, vo = O.prefill(w, cfg, O.bf16_to_f64(bits), np.arange(T), W=W)
    assert_parity(y.cpu().numpy(), yo, "y")
    assert_parity(cache_values(k)[0][:, L:L + T].transpose(1, 0, 2), ko, "new K")
    assert_parity(cache_values(v)[0][:, L:L + T].transpose(1, 0, 2), vo, "new V")
