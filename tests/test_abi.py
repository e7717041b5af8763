"""C-ABI checks that need no GPU: the library loads, exports every entry point the
header declares, sizes its workspaces, and rejects bad arguments before enqueueing
anything (all calls here fail validation or are no-ops, so no kernel is launched)."""
import ctypes
import os
import re

import pytest

from paper_2609_24433_amd import fq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "fq.h")

NULL = None
FAKE = ctypes.c_void_p(0x10000)  # never dereferenced: every call below fails validation first
MISALIGNED = ctypes.c_void_p(0x10004)


def declared_symbols():
    text = open(HEADER).read()
    return sorted(set(re.findall(r"^\s*(?:const\s+)?[a-z_0-9]+\s*\*?\s*(fq_[a-z0-9_]+)\s*\(", text, re.M)))


def test_header_declares_the_boundary():
    syms = declared_symbols()
    assert set(syms) == set(fq.EXPORTED), syms


@pytest.mark.parametrize("name", declared_symbols())
def test_library_exports_symbol(name):
    assert hasattr(fq.LIB, name)


def test_status_strings():
    for s in range(8):
        assert fq.LIB.fq_status_string(s) not in (None, b"", b"unknown status")
    assert fq.LIB.fq_status_string(99) == b"unknown status"


def test_sizes():
    assert fq.packed_weight_bytes(2048, 16384, 4) == 2048 * 16384 // 2
    assert fq.packed_weight_bytes(2048, 16384, 8) == 2048 * 16384
    assert fq.packed_weight_bytes(16, 128, 3) == 0
    assert fq.gemm_workspace_bytes(0, 16, 128, 4) == 0
    # linear workspace holds the intermediate codes (nibbles for W4A4, int8 for W8A8), the
    # token scales and the GEMM's own workspace
    for bits in (4, 8):
        assert fq.linear_workspace_bytes(50, 2048, 16384, bits) >= (
            50 * 16384 * bits // 8 + 50 * 4 + fq.gemm_workspace_bytes(50, 2048, 16384, bits))
    for M in (1, 16, 50, 64, 65, 816, 4096):
        assert fq.gemm_workspace_bytes(M, 2048, 16384, 4) % 256 == 0


def _a256(n):
    return (n + 255) // 256 * 256


def test_plan_workspaces():
    """The workspaces pin the launch plans of the long-K W4A4 projection (K 16384 -> N 2048):
    the k-group GEMM needs no split-K partials; the GEMM entry point feeds it a k-major copy of
    the canonical codes (M = 816), the fused projection's prologue writes that order itself (M =
    816 to 2048, and for the wide tiles 3072 and 4096); M = 2048 and 4096 through the GEMM entry
    point take the LDS-ring kernel unsplit."""
    K, N = 16384, 2048
    assert fq.gemm_workspace_bytes(816, N, K, 4) == _a256(816 * K // 2)
    for M in (2048, 4096):
        assert fq.gemm_workspace_bytes(M, N, K, 4) == 0
    for M in (816, 1600, 2048, 3072, 4096):
        assert fq.linear_workspace_bytes(M, N, K, 4) == _a256(M * K // 2) + _a256(M * 4)
    # W8A8 at M = 816 splits K in two: int32 partials [2][M][N]
    assert fq.gemm_workspace_bytes(816, N, K, 8) == _a256(2 * 816 * N * 4)


def call_quant(x=FAKE, ldx=1024, smooth=NULL, M=4, K=1024, b=64, bits=4, r=1.0, codes=FAKE, delta=FAKE,
               post=NULL):
    return fq.LIB.fq_fwht_quant(x, ldx, smooth, post, M, K, b, bits, r, codes, delta, None)


@pytest.mark.parametrize("kw,status", [
    (dict(x=NULL), 1), (dict(codes=NULL), 1), (dict(delta=NULL), 1),
    (dict(M=-1), 2), (dict(ldx=1000), 2), (dict(b=128, K=1024 + 128 + 64), 3),
    (dict(K=1024 + 64), 3), (dict(K=64), 3), (dict(K=65536), 3),
    (dict(b=3), 3), (dict(b=512), 3), (dict(b=0), 3), (dict(bits=2), 3), (dict(bits=16), 3),
    (dict(r=0.0), 3), (dict(r=1.5), 3), (dict(r=float("nan")), 3),
    (dict(x=MISALIGNED), 4), (dict(codes=MISALIGNED), 4), (dict(ldx=1028), 4),
    (dict(smooth=MISALIGNED), 4), (dict(post=MISALIGNED), 4),
])
def test_fwht_quant_rejects(kw, status):
    assert call_quant(**kw) == status
    assert fq.LIB.fq_last_error()


def test_fwht_quant_k_not_multiple_of_b():
    assert call_quant(K=1152, ldx=1152, b=256) == 2


def test_zero_rows_are_noops():
    assert call_quant(M=0, x=NULL, codes=NULL, delta=NULL) == 0
    assert fq.LIB.fq_gemm_w4a4(NULL, NULL, NULL, NULL, NULL, NULL, 16, NULL, 0, 16, 128, NULL, 0, None) == 0
    assert fq.LIB.fq_linear(NULL, 1024, NULL, NULL, 0, 1024, 256, 64, 4, 1.0, NULL, NULL, NULL, NULL, 256, NULL,
                            0, None) == 0


def call_gemm(bits=4, a=FAKE, delta=FAKE, w=FAKE, sw=FAKE, bias=NULL, y=FAKE, ldy=256, acc=NULL,
              M=50, N=256, K=1024, ws=FAKE, ws_bytes=1 << 30):
    fn = fq.LIB.fq_gemm_w4a4 if bits == 4 else fq.LIB.fq_gemm_w8a8
    return fn(a, delta, w, sw, bias, y, ldy, acc, M, N, K, ws, ws_bytes, None)


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("kw,status", [
    (dict(a=NULL), 1), (dict(delta=NULL), 1), (dict(w=NULL), 1), (dict(sw=NULL), 1), (dict(y=NULL), 1),
    (dict(M=-3), 2), (dict(ldy=128), 2), (dict(N=-16), 2),
    (dict(N=250, ldy=256), 3), (dict(K=1000), 3), (dict(K=0), 3),
    (dict(M=1 << 24, N=1 << 20, ldy=1 << 20), 3),  # more outputs than the launch grids index
    (dict(bias=MISALIGNED), 4), (dict(acc=MISALIGNED), 4), (dict(ldy=260), 4), (dict(w=MISALIGNED), 4),
    (dict(ws=NULL, ws_bytes=0, M=50, N=2048, ldy=2048, K=32768), 5),
    (dict(ws_bytes=16, M=50, N=2048, ldy=2048, K=32768), 5),
])
def test_gemm_rejects(bits, kw, status):
    if status == 5:
        # the shape must split K (need a workspace), or the call would go on to launch
        assert fq.gemm_workspace_bytes(kw["M"], kw["N"], kw["K"], bits) > 16
    assert call_gemm(bits=bits, **kw) == status


def call_linear(x=FAKE, ldx=1024, M=50, K=1024, N=256, b=64, bits=4, r=1.0, w=FAKE, sw=FAKE, bias=NULL,
                y=FAKE, ldy=256, ws=FAKE, ws_bytes=1 << 30, smooth=NULL, post=NULL):
    return fq.LIB.fq_linear(x, ldx, smooth, post, M, K, N, b, bits, r, w, sw, bias, y, ldy, ws, ws_bytes, None)


@pytest.mark.parametrize("kw,status", [
    (dict(x=NULL), 1), (dict(w=NULL), 1), (dict(y=NULL), 1), (dict(sw=NULL), 1),
    (dict(ldx=512), 2), (dict(ldy=100), 2), (dict(b=5), 3), (dict(bits=6), 3), (dict(N=40, ldy=40), 3),
    (dict(r=-1.0), 3), (dict(smooth=MISALIGNED), 4), (dict(post=MISALIGNED), 4),
    # shapes that need a workspace (too long for the one-kernel path)
    (dict(ws=NULL, ws_bytes=0, K=16384, ldx=16384), 5), (dict(ws_bytes=100, K=16384, ldx=16384), 5),
    (dict(ws=MISALIGNED, K=16384, ldx=16384), 4),
])
def test_linear_rejects(kw, status):
    if status in (4, 5) and "ws" in kw or "ws_bytes" in kw:
        assert fq.linear_workspace_bytes(kw.get("M", 50), kw.get("N", 256), kw["K"], kw.get("bits", 4)) > 100
    assert call_linear(**kw) == status


@pytest.mark.parametrize("fn", ["fq_pack_weights", "fq_unpack_weights"])
def test_pack_rejects(fn):
    f = getattr(fq.LIB, fn)
    assert f(NULL, 32, 128, 4, FAKE, None) == 1
    assert f(FAKE, 30, 128, 4, FAKE, None) == 3
    assert f(FAKE, 32, 100, 4, FAKE, None) == 3
    assert f(FAKE, 32, 128, 5, FAKE, None) == 3
    assert f(FAKE, -16, 128, 4, FAKE, None) == 2
    assert f(MISALIGNED, 32, 128, 4, FAKE, None) == 4
    assert f(FAKE, 0, 128, 4, FAKE, None) == 0


def test_quantize_weights_rejects():
    f = fq.LIB.fq_quantize_weights
    assert f(NULL, 128, NULL, NULL, 16, 128, 64, 4, FAKE, FAKE, None) == 1
    assert f(FAKE, 130, NULL, NULL, 16, 128, 64, 4, FAKE, FAKE, None) == 4
    assert f(FAKE, 64, NULL, NULL, 16, 128, 64, 4, FAKE, FAKE, None) == 2
    assert f(FAKE, 128, NULL, NULL, 16, 128, 64, 7, FAKE, FAKE, None) == 3
    assert f(FAKE, 128, NULL, MISALIGNED, 16, 128, 64, 4, FAKE, FAKE, None) == 4


def call_w4a16(x=FAKE, ldx=1024, w=FAKE, sw=FAKE, bias=NULL, y=FAKE, ldy=256, acc=NULL, M=1, N=256, K=1024,
               ws=FAKE, ws_bytes=1 << 30):
    return fq.LIB.fq_gemm_w4a16(x, ldx, w, sw, bias, y, ldy, acc, M, N, K, ws, ws_bytes, None)


@pytest.mark.parametrize("kw,status", [
    (dict(x=NULL), 1), (dict(w=NULL), 1), (dict(sw=NULL), 1), (dict(y=NULL), 1),
    (dict(M=-1), 2), (dict(ldx=512), 2), (dict(ldy=128), 2),
    (dict(N=250, ldy=256), 3), (dict(K=1000, ldx=1000), 3), (dict(K=0), 3),
    (dict(M=1 << 23, N=16, ldy=16), 3),  # more 64-row blocks than the grid's z dimension holds
    (dict(x=MISALIGNED), 4), (dict(acc=MISALIGNED), 4), (dict(ldx=1028), 4), (dict(bias=MISALIGNED), 4),
    (dict(ws=NULL, ws_bytes=0, K=32768, ldx=32768), 5), (dict(ws_bytes=8, K=32768, ldx=32768), 5),
])
def test_w4a16_rejects(kw, status):
    if status == 5:
        # the shape must split K (need a workspace), or the call would go on to launch
        assert fq.w4a16_workspace_bytes(kw.get("M", 1), kw.get("N", 256), kw["K"]) > 8
    assert call_w4a16(**kw) == status


def test_w4a16_workspace_sizes():
    assert fq.w4a16_workspace_bytes(1, 2048, 1024) == 0          # one K slice: no partials
    assert fq.w4a16_workspace_bytes(1, 2048, 8192) == 0          # a single token up to K = 8192
    assert fq.w4a16_workspace_bytes(1, 2048, 16384) >= 4 * 1 * 2048 * 4
    assert fq.w4a16_workspace_bytes(2, 2048, 16384) >= 4 * 2 * 2048 * 4
    assert fq.w4a16_workspace_bytes(0, 2048, 16384) == 0
    assert call_w4a16(M=0, x=NULL, w=NULL, sw=NULL, y=NULL) == 0


def call_rotate(x=FAKE, ldx=1024, perm=NULL, blocks=FAKE, smooth=NULL, post=NULL, M=4, K=1024, b=64, bits=4,
                r=1.0, codes=FAKE, delta=FAKE, ws=FAKE, ws_bytes=1 << 30):
    return fq.LIB.fq_rotate_quant(x, ldx, perm, blocks, smooth, post, M, K, b, bits, r, codes, delta, ws,
                                  ws_bytes, None)


@pytest.mark.parametrize("kw,status", [
    (dict(x=NULL), 1), (dict(blocks=NULL), 1), (dict(codes=NULL), 1), (dict(delta=NULL), 1),
    (dict(M=-1), 2), (dict(ldx=512), 2), (dict(K=1024 + 128, b=256, ldx=1152), 2),
    (dict(b=256), 3), (dict(b=48), 3), (dict(K=65536, ldx=65536), 3), (dict(bits=3), 3), (dict(r=0.0), 3),
    (dict(perm=MISALIGNED), 4), (dict(blocks=MISALIGNED), 4), (dict(post=MISALIGNED), 4), (dict(ldx=1028), 4),
    (dict(ws=NULL, ws_bytes=0), 5), (dict(ws_bytes=4 * 4 * 1024 - 1), 5), (dict(ws=MISALIGNED), 4),
])
def test_rotate_quant_rejects(kw, status):
    assert call_rotate(**kw) == status


def test_rotate_quant_workspace_and_empty():
    assert fq.LIB.fq_rotate_quant_workspace_bytes(4, 1024) >= 4 * 1024 * 4
    assert fq.LIB.fq_rotate_quant_workspace_bytes(0, 1024) == 0
    assert call_rotate(M=0, x=NULL, blocks=NULL, codes=NULL, delta=NULL, ws=NULL, ws_bytes=0) == 0
    # the weight side takes fp32 rows: a leading dimension that is a multiple of 4 suffices
    assert fq.LIB.fq_quantize_weights_rotated(FAKE, 1028, NULL, NULL, NULL, NULL, 16, 1024, 64, 4, FAKE, FAKE,
                                              FAKE, 1 << 30, None) == 1


@pytest.mark.parametrize("call,status", [
    (lambda: fq.LIB.fq_transform(NULL, 0, 1024, NULL, NULL, 4, 1024, 64, FAKE, None), 1),
    (lambda: fq.LIB.fq_transform(FAKE, 0, 1024, NULL, NULL, 4, 1024, 512, FAKE, None), 3),
    (lambda: fq.LIB.fq_transform(FAKE, 1, 1026, NULL, NULL, 4, 1024, 64, FAKE, None), 4),
    (lambda: fq.LIB.fq_gptq_hessian(FAKE, 1024, 8, 1000, FAKE, 0, None), 3),
    (lambda: fq.LIB.fq_gptq_hessian(FAKE, 1024, 8, 32768, FAKE, 0, None), 3),
    (lambda: fq.LIB.fq_gptq_hessian(FAKE, 512, 8, 1024, FAKE, 0, None), 2),
    (lambda: fq.LIB.fq_gptq_hessian(FAKE, 1024, 8, 1024, NULL, 0, None), 1),
    (lambda: fq.LIB.fq_gptq_factor(FAKE, 1024, 2.0, FAKE, FAKE, 1 << 40, None), 3),
    (lambda: fq.LIB.fq_gptq_factor(FAKE, 1024, 0.01, FAKE, FAKE, 8, None), 5),
    (lambda: fq.LIB.fq_gptq_factor(FAKE, 1024, 0.01, MISALIGNED, FAKE, 1 << 40, None), 4),
    (lambda: fq.LIB.fq_gptq_sweep(FAKE, 1024, FAKE, 16, 1024, 128, 3, FAKE, FAKE, FAKE, 1 << 40, None), 3),
    (lambda: fq.LIB.fq_gptq_sweep(FAKE, 1000, FAKE, 16, 1024, 128, 4, FAKE, FAKE, FAKE, 1 << 40, None), 2),
    (lambda: fq.LIB.fq_gptq_sweep(FAKE, 1024, NULL, 16, 1024, 128, 4, FAKE, FAKE, FAKE, 1 << 40, None), 1),
    (lambda: fq.LIB.fq_gptq_sweep(FAKE, 1024, FAKE, 16, 1024, 48, 4, FAKE, FAKE, FAKE, 1 << 40, None), 3),
    (lambda: fq.LIB.fq_gptq_sweep(FAKE, 1024, FAKE, 16, 1024, 512, 4, FAKE, FAKE, FAKE, 1 << 40, None), 3),
    (lambda: fq.LIB.fq_gptq_sweep(FAKE, 1024, FAKE, 16, 1024, 128, 4, FAKE, FAKE, FAKE, 64, None), 5),
    (lambda: fq.LIB.fq_gptq_sweep(FAKE, 1024, FAKE, 0, 1024, 128, 4, NULL, NULL, NULL, 0, None), 0),
])
def test_gptq_rejects(call, status):
    assert call() == status


def test_gptq_workspace_sizes():
    assert fq.LIB.fq_gptq_factor_workspace_bytes(1024) >= 2 * 1024 * 1024 * 8
    assert fq.LIB.fq_gptq_factor_workspace_bytes(32768) == 0
    assert fq.LIB.fq_gptq_sweep_workspace_bytes(64, 1024) >= 64 * 1024 * 8
    assert fq.LIB.fq_gptq_sweep_workspace_bytes(0, 1024) == 0


# ---- K outside whole 128-channel steps (the weight tiles' width) is rejected everywhere ----

@pytest.mark.parametrize("K", [32, 96, 160, 1024 + 32])
def test_k_not_whole_steps_rejected(K):
    b = 32
    assert call_quant(K=K, ldx=max(K, 1024), b=b) == 3
    for bits in (4, 8):
        assert call_gemm(bits=bits, K=K) == 3
    assert call_linear(K=K, ldx=max(K, 1024), b=b) == 3
    assert fq.LIB.fq_pack_weights(FAKE, 32, K, 4, FAKE, None) == 3
    assert call_w4a16(K=K, ldx=max(K, 1024)) == 3
    assert "multiple of 128" in fq.LIB.fq_last_error().decode() or "outside" in fq.LIB.fq_last_error().decode()


# ---- outputs may not overlap inputs or each other (FQ_ERR_ALIAS = 7) ----

BASE = 1 << 24  # fake, never dereferenced addresses: these calls fail validation


def _ptr(off):
    return ctypes.c_void_p(BASE + off)


def test_fwht_quant_alias_rejected():
    # x rows [BASE, BASE + 4 * 2048); codes inside them
    assert call_quant(x=_ptr(0), codes=_ptr(1024), delta=_ptr(1 << 20)) == 7
    assert call_quant(x=_ptr(0), codes=_ptr(1 << 20), delta=_ptr((1 << 20) + 256)) == 7   # codes and delta
    assert call_quant(x=_ptr(0), codes=_ptr(1 << 20), delta=_ptr(2 << 20), smooth=_ptr((2 << 20) - 16)) == 7


def test_gemm_alias_rejected():
    # y overlaps the codes; acc overlaps y; the workspace overlaps the weights
    assert call_gemm(a=_ptr(0), y=_ptr(256), delta=_ptr(1 << 20), w=_ptr(2 << 20), sw=_ptr(3 << 20)) == 7
    assert call_gemm(a=_ptr(0), y=_ptr(1 << 20), acc=_ptr((1 << 20) + 4096), delta=_ptr(2 << 20),
                     w=_ptr(3 << 20), sw=_ptr(4 << 20)) == 7
    assert call_gemm(M=50, N=2048, ldy=2048, K=32768, a=_ptr(0), y=_ptr(4 << 20), delta=_ptr(5 << 20),
                     w=_ptr(8 << 20), sw=_ptr(6 << 20), ws=_ptr(9 << 20)) == 7


def test_linear_alias_rejected():
    # the workspace overlaps y (a shape that needs one); y overlaps x
    assert fq.linear_workspace_bytes(50, 256, 16384, 4) > 0
    assert call_linear(K=16384, ldx=16384, x=_ptr(0), y=_ptr(4 << 20), ws=_ptr((4 << 20) + 4096),
                       w=_ptr(8 << 20), sw=_ptr(3 << 20)) == 7
    assert call_linear(x=_ptr(0), y=_ptr(2048), ws=_ptr(4 << 20), w=_ptr(2 << 20), sw=_ptr(3 << 20)) == 7
    assert call_linear(x=_ptr(0), y=_ptr(1 << 20), ws=NULL, ws_bytes=0, w=_ptr((1 << 20) + 64),
                       sw=_ptr(3 << 20)) == 7  # y overlaps the weights


def test_gptq_and_transform_alias_rejected():
    assert fq.LIB.fq_transform(_ptr(0), 1, 1024, NULL, NULL, 4, 1024, 64, _ptr(4096), None) == 7
    assert fq.LIB.fq_gptq_hessian(_ptr(0), 1024, 8, 1024, _ptr(1024), 0, None) == 7


# ---- no development override is read by the shipped library ----

def test_library_reads_no_tuning_environment():
    with open(fq.LIB_PATH, "rb") as f:
        blob = f.read()
    assert b"FQ_TUNE" not in blob
    assert b"getenv" not in blob


# ---- the binding checks caller-supplied outputs before calling the library ----

def test_binding_rejects_mismatched_outputs():
    import torch
    codes = torch.zeros((4, 512), dtype=torch.uint8)
    delta = torch.zeros((4,), dtype=torch.float32)
    w = torch.zeros((16 * 512,), dtype=torch.uint8)
    sw = torch.zeros((16,), dtype=torch.float32)
    for bad in (torch.empty((4, 16), dtype=torch.float32), torch.empty((4, 32), dtype=torch.bfloat16),
                torch.empty((16, 4), dtype=torch.bfloat16).t()):
        with pytest.raises(ValueError):
            fq.gemm(codes, delta, w, sw, 16, 1024, 4, out=bad)
    with pytest.raises(ValueError):
        fq.gemm(torch.zeros((4, 1024), dtype=torch.uint8), delta, w, sw, 16, 1024, 4)  # int8-wide codes for W4A4
    x = torch.zeros((4, 1024), dtype=torch.bfloat16)
    with pytest.raises(ValueError):
        fq.linear(x, w, sw, 16, 64, 4, out=torch.empty((4, 16), dtype=torch.float16))
    with pytest.raises(ValueError):
        fq.fwht_quant(x, 64, 4, out_codes=torch.empty((4, 1024), dtype=torch.uint8))


def test_linear_static_rejects_before_any_device_call():
    """The scratch limit and the argument checks come before the library touches a device."""
    f = fq.LIB.fq_linear_static
    assert fq.LIB.fq_linear_static_max_workspace_bytes() == 64 << 20
    assert fq.linear_workspace_bytes(4096, 2048, 32768, 8) > 64 << 20
    assert f(FAKE, 32768, NULL, NULL, 4096, 32768, 2048, 128, 8, 1.0, FAKE, FAKE, NULL, FAKE, 2048, None) == 5
    assert b"fq_linear_static holds" in fq.LIB.fq_last_error()
    assert f(NULL, 1024, NULL, NULL, 4, 1024, 256, 64, 4, 1.0, FAKE, FAKE, NULL, FAKE, 256, None) == 1
    assert f(FAKE, 1024, NULL, NULL, 4, 1000, 256, 64, 4, 1.0, FAKE, FAKE, NULL, FAKE, 256, None) == 3
    assert f(NULL, 1024, NULL, NULL, 0, 1024, 256, 64, 4, 1.0, NULL, NULL, NULL, NULL, 256, None) == 0
