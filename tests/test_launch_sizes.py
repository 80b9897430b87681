"""Size arithmetic of the decode GEMV's launches on the host, no GPU needed, at
the largest shapes that layer_create accepts."""
import ctypes

import pytest

from paper_2607_15865_amd import binding as B

WF = {"int4": 0, "int8": 1, "f16": 2}
PAST_END = 0xFFFF0000                            # offset of the loads that must return 0


def run_bytes(tile, ct, K_pad, wf):
    first, nbytes = ctypes.c_uint64(), ctypes.c_uint32()
    B._lib.w4_gemv_run_bytes(tile, ct, K_pad, WF[wf], ctypes.byref(first), ctypes.byref(nbytes))
    return first.value, nbytes.value


@pytest.mark.parametrize("K,N,wf", [
    (16384, 131072, "f16"),                      # gate/up of hidden 16384, FFN 65536: 2^32 bytes
    (16384, 131072, "int8"), (16384, 131072, "int4"), (65536, 16384, "f16"), (128, 256, "int4"),
    (16384, 262144, "f16")])                     # beyond 2^32 bytes
@pytest.mark.parametrize("ct", [1, 2])
def test_gemv_blocks_cover_the_matrix(K, N, wf, ct):
    """The blocks' weight runs are not empty, follow each other without a gap, end
    with the matrix, and end below the offset that stands for "past the end"."""
    total = K * N * {"int4": 1, "int8": 2, "f16": 4}[wf] // 2
    end = 0
    for tile in range(0, N // 32, ct):
        first, nbytes = run_bytes(tile, ct, K, wf)
        assert first == end and nbytes == ct * 32 * K * total // (K * N)
        end = first + nbytes
    assert end == total
    assert nbytes <= 1 << 25 and nbytes < PAST_END
