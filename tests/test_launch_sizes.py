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


def resid_plan(B_, K, N, zp=False, group=128, ordered=False, cus=256):
    ks, lds = ctypes.c_int(), ctypes.c_uint64()
    B._lib.w4_gemv_resid_plan(B_, K, N, int(zp), group.bit_length() - 1, int(ordered), cus, ctypes.byref(ks), ctypes.byref(lds))
    return ks.value, lds.value


@pytest.mark.parametrize("zp,group", [(False, 128), (True, 128), (False, 32), (True, 32)])
def test_residual_gemvs_fit_the_lds(zp, group):
    """Every width and depth that layer_create accepts gets k ranges whose rows and
    corrections fit a CU's 160 KB, at every batch; ranges stay whole k tiles."""
    for N in range(128, 16385, 128):
        for K in (128, 2048, 14336, 28672, 32768, 40960, 53248, 57344, 61440, 65536):
            for rows in range(1, 9):
                ks, lds = resid_plan(rows, K, N, zp, group)
                assert 1 <= ks <= K // 64 and lds <= 160 * 1024, (N, K, rows, ks, lds)


def test_ordered_residual_gemvs_take_at_most_two_ranges():
    """(Adds of two ranges onto 0 commute; one or two rows of the depths that the
    persistent launch, whose place they take, can hold.)"""
    for N in range(512, 16385, 128):
        for K, rows in ((65536, 1), (40960, 1), (32768, 2), (32768, 1), (14336, 2), (512, 2)):
            ks, lds = resid_plan(rows, K, N, ordered=True)
            assert ks <= 2 and lds <= 160 * 1024, (N, K, rows, ks, lds)
