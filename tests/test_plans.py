"""Which GEMM the planner takes (no GPU needed): the lines of the wide-tile and the k-group kernels,
with a shape on each side, and the scratch that comes with them."""
import ctypes

import pytest
import torch

from paper_2609_24433_amd import fq

LDS_RING, KGROUP, WIDE = 1, 3, 4


class _Plan(ctypes.Structure):
    # the plan's first member is its kind; the rest is room for the callee to fill
    _fields_ = [("kind", ctypes.c_int), ("rest", ctypes.c_byte * 252)]


_plan_gemm = fq.LIB["_ZN2fq9plan_gemmElllib"]  # fq::plan_gemm(long, long, long, int, bool)
_plan_gemm.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_bool]
_plan_gemm.restype = _Plan


def kind(M, K, N, bits, fused=True):
    return _plan_gemm(M, N, K, bits, fused).kind


@pytest.mark.parametrize("M,K,N,bits,want", [
    # rows past M: 128 rows fill half of a 256-row tile, which takes twice as many rounds
    (128, 2048, 65536, 4, LDS_RING), (128, 2048, 65536, 8, LDS_RING), (65, 4096, 33280, 4, LDS_RING),
    (100, 4096, 36864, 8, LDS_RING), (256, 2048, 33280, 4, WIDE), (256, 2048, 33280, 8, WIDE),
    (807, 4352, 9200, 4, LDS_RING), (382, 2176, 17040, 8, LDS_RING),
    (816, 2048, 32768, 4, WIDE), (816, 2048, 16384, 8, WIDE), (257, 2048, 16384, 4, WIDE),
    (4096, 16384, 2048, 4, WIDE), (4096, 16384, 2048, 8, WIDE),
    # a few more rounds from a longer K on: 3 against 2, 4 against 3, 6 against 5
    (383, 2944, 32896, 4, LDS_RING), (383, 3072, 32896, 4, WIDE), (383, 3456, 32896, 8, LDS_RING),
    (383, 3584, 32896, 8, WIDE), (831, 1664, 25600, 4, LDS_RING), (831, 1792, 25600, 4, WIDE),
    (831, 384, 25600, 8, LDS_RING), (831, 512, 25600, 8, WIDE),
    (1647, 1280, 24320, 4, LDS_RING), (1647, 1408, 24320, 4, WIDE), (1647, 128, 24320, 8, WIDE),
    # short K: one round, two, three
    (2048, 256, 4096, 4, LDS_RING), (2048, 384, 4096, 4, WIDE), (2048, 128, 4096, 8, WIDE),
    (2277, 896, 4992, 4, LDS_RING), (2277, 1024, 4992, 4, WIDE),
    (2277, 384, 4992, 8, LDS_RING), (2277, 512, 4992, 8, WIDE),
    (3041, 512, 5168, 4, LDS_RING), (3041, 640, 5168, 4, WIDE), (3041, 128, 5168, 8, WIDE),
    (1280, 384, 9872, 8, WIDE), (1280, 384, 9344, 8, LDS_RING),
    (3078, 128, 7360, 8, WIDE),
    # one 128 x 128 tile per compute unit
    (2048, 2048, 2048, 8, LDS_RING), (2048, 2048, 2064, 8, WIDE),
])
def test_wide_tiles(M, K, N, bits, want):
    assert kind(M, K, N, bits) == want
    if bits == 8:
        assert kind(M, K, N, bits, fused=False) == want
    else:
        assert kind(M, K, N, bits, fused=False) != WIDE


@pytest.mark.parametrize("M,K,N,want", [
    (65, 4096, 256, KGROUP), (512, 4096, 4096, KGROUP), (512, 3968, 4096, LDS_RING), (512, 4096, 4160, LDS_RING),
    (3968, 4224, 512, LDS_RING), (3968, 4224, 384, KGROUP), (3200, 4224, 512, KGROUP),
    # from K = 8192 on the LDS-ring kernel's split K has the grids of up to 64 tiles of 128 x 128
    (128, 8192, 3072, LDS_RING), (358, 9088, 816, LDS_RING), (384, 16384, 2048, LDS_RING), (256, 24576, 3840, LDS_RING),
    (801, 16512, 1040, LDS_RING), (1024, 16384, 1024, LDS_RING), (640, 11520, 1568, KGROUP), (801, 16512, 1200, KGROUP),
    (816, 16384, 2048, KGROUP), (1600, 16384, 2048, KGROUP), (2048, 16384, 2048, KGROUP), (1327, 9088, 1792, KGROUP),
    (785, 8192, 4240, LDS_RING), (785, 9216, 4240, KGROUP),
])
def test_k_groups(M, K, N, want):
    assert kind(M, K, N, 4) == want


def test_small_grids_of_long_rows_fit_the_static_scratch():
    """A small grid whose split K would need more scratch than fq_linear_static holds is served without
    partial sums: the call gets past its scratch check (and ends at the missing device here)."""
    limit = fq.LIB.fq_linear_static_max_workspace_bytes()
    fake = ctypes.c_void_p(0x10000)
    tried = 0
    for K in range(8192, 32769, 1024):
        for N in (80, 128, 256):
            M = ((limit - 65536) * 2 // K) // 128 * 128
            if M // 128 * ((N + 127) // 128) <= 64 and (M // 128) * ((N + 63) // 64) >= (48 if K < 16384 else 96):
                assert kind(M, K, N, 4) == LDS_RING and fq.linear_workspace_bytes(M, N, K, 4) > limit
                if not torch.cuda.is_available():
                    y, w = ctypes.c_void_p(1 << 40), ctypes.c_void_p(1 << 41)
                    rc = fq.LIB.fq_linear_static(ctypes.c_void_p(1 << 42), K, None, None, M, K, N, 128, 4, 1.0, w, fake,
                                                 None, y, (N + 7) // 8 * 8, None)
                    assert rc == 6, fq.LIB.fq_last_error()
                tried += 1
    assert tried > 5
