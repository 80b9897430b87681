"""The first calls of a process: the kernels' code is loaded when the layer is
created, not by the first call that needs it (9 ms for the first prefill, 3 ms for
the first decode step, when the runtime loaded it then; 0.7 and 0.1 ms since)."""
import os
import subprocess
import sys

import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu

CHILD = """
import time
import torch
from paper_2607_15865_amd import binding, synth
cfg = synth.CONFIGS["tiny"]
lay = binding.Layer(cfg, synth.make_layer(cfg))
k, v = lay.new_cache(1, 0)
x, pos = torch.randn((64, cfg.hidden), device="cuda"), torch.arange(64, dtype=torch.int32, device="cuda")
y, c = torch.zeros_like(x), pos[40:41].clone()
x1, y1 = x[:1].clone(), y[:1].clone()
torch.cuda.synchronize()
t = time.perf_counter()
lay.prefill(x, pos, k, v, y)
lay.set_decode_path(1)
lay.decode(x1, c, c, 40, k, v, y1)
torch.cuda.synchronize()
print((time.perf_counter() - t) * 1e3)
"""


def test_first_calls_load_no_code():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    times = []
    for _ in range(3):                           # (a busy host may slow one of them)
        r = subprocess.run([sys.executable, "-c", CHILD], cwd=root, capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stderr
        times.append(float(r.stdout.split()[-1]))
        log(f"first prefill and decode of a process: {times[-1]:.2f} ms")
        if times[-1] < 3.0:
            return
    assert False, times
