"""The k-major codes that the fused INT4 projection's prologue writes for the k-group and the
wide-tile GEMM, against the canonical codes of the two separate entry points: the outputs are equal
bit for bit."""
import pytest
import torch

import tests.test_gpu_wide as wide
from paper_2609_24433_amd import synth
from tests.gpu_util import DEV, flush

pytestmark = pytest.mark.gpu

KGROUP, WIDE = (333, 6272, 1552), (257, 2048, 16400)  # M, K, N that take these kernels


def both_paths(x, w, b, bits, clip=1.0, s=None, p=None):
    """The fused projection and the prologue + GEMM on the same tokens, as bit patterns."""
    from paper_2609_24433_amd import fq
    M, K = x.shape
    N = w.shape[0]
    wc, sw = fq.quantize_weights(w, b, bits, s, p)
    wp = fq.pack_weights(wc, bits)
    pre, post = (None if v is None else 1.0 / v for v in (s, p))
    y = fq.linear(x, wp, sw, N, b, bits, clip, pre, post_inv=post)
    codes, delta = fq.fwht_quant(x, b, bits, clip, pre, post_inv=post)
    y2 = fq.gemm(codes, delta, wp, sw, N, K, bits)
    torch.cuda.synchronize()
    return y.view(torch.int16), y2.view(torch.int16)


@pytest.mark.parametrize("M,K,N", [KGROUP, WIDE])
@pytest.mark.parametrize("clip", [1.0, 0.9])
@pytest.mark.parametrize("value", [float("nan"), -float("nan"), float("inf"), -float("inf")])
def test_tokens_that_are_not_finite(M, K, N, clip, value):
    """A NaN or an infinity in a token spoils its own block's codes as on the other path (code -8 for a
    NaN) and no other channel's."""
    flush(f"major codes of {value} M={M} K={K} N={N} clip={clip}")
    x = synth.activations(M, K, seed=M, outlier_frac=0.01, outlier_scale=30.0)
    for c in range(48):  # every place of a chunk, one row each
        x[3 + 5 * c, 1000 + c] = value
    w = torch.from_numpy(synth.weights(N, K, seed=N)).to(DEV)
    for b in (1, 32):
        y, y2 = both_paths(x.to(DEV), w, b, 4, clip)
        assert torch.equal(y, y2)


@pytest.mark.parametrize("b", [1, 32, 128, 256])
@pytest.mark.parametrize("clip,folds", [(0.9, "both"), (0.75, "none"), (1.0, "before"), (1.0, "after")])
@pytest.mark.parametrize("M,K,N", [
    # the k groups and the wide tiles from every row shape of the prologue: rows that share a workgroup
    # (K up to 4096), 256, 512 and 1024 threads a row
    (333, 4096, 1552), (333, 6144, 1552), (801, 16384, 1552), (700, 32768, 1552), (257, 2048, 16400), (2049, 1024, 2064)])
def test_folds_clips_and_blocks(M, K, N, b, clip, folds):
    flush(f"major codes M={M} K={K} N={N} b={b} clip={clip} folds={folds}")
    x = synth.activations(M, K, seed=M + b, outlier_frac=0.01, outlier_scale=30.0).to(DEV)
    w = torch.from_numpy(synth.weights(N, K, seed=N)).to(DEV)
    vec = lambda seed, on: torch.from_numpy(synth.channel_vector(K, seed=seed, low=0.5, high=2.0)).to(DEV) if on else None
    y, y2 = both_paths(x, w, b, 4, clip, vec(1, folds in ("before", "both")), vec(2, folds in ("after", "both")))
    assert torch.equal(y, y2)


# two k steps (INT8), k steps that are 2 mod 4 (both widths)
@pytest.mark.parametrize("M,K,N,bits", [(300, 256, 12304, 8), (2049, 768, 2064, 4), (2049, 768, 2064, 8),
                                        (1000, 1280, 4240, 4), (1000, 1280, 4240, 8)])
def test_wide_tiles_k_steps(M, K, N, bits):
    wide.test_fused_equals_split(M, K, N, bits)


@pytest.mark.parametrize("M,N", [(816, 2048), (2064, 2064)])  # the k groups, the wide tiles
def test_long_sums_to_the_last_unit(M, N):
    """K = 32768 of codes 5 to 7: the products' fp32 sums of (code + 8) reach 7 million with all their low
    bits in use.  A row differs from row 0 in at most 20 codes by one, and the bias takes row 0's sum
    off before the bf16 rounding, so what is left is an integer below 256, which bf16 holds: an error
    of one unit in an accumulator shows."""
    from paper_2609_24433_amd import fq
    K = 32768
    flush(f"long sums M={M} N={N}")
    g = torch.Generator().manual_seed(M)
    w = torch.randint(5, 8, (N, K), generator=g)
    base = torch.randint(5, 8, (K,), generator=g)
    w[:, 0] = base[0] = 7  # every row's maximum: its step is 1
    step = torch.zeros((M, K), dtype=torch.int64)
    at = torch.randint(1, K, (M, 20), generator=g)
    step.scatter_(1, at, torch.where(base[at] == 7, -1, 1) * (torch.arange(20) < 10 + torch.arange(M)[:, None] % 11))
    step[0] = 0
    x = (base + step).to(torch.bfloat16).to(DEV)
    wc, sw = fq.quantize_weights(w.float().to(DEV), 1, 4)
    assert torch.equal(wc.cpu().long(), w) and bool((sw == 1).all())
    sum0 = (w.double() @ base.double()).long()
    y = fq.linear(x, fq.pack_weights(wc, 4), sw, N, 1, 4, bias=-sum0.float().to(DEV))
    want = (step.double().to(DEV) @ w.double().to(DEV).t().contiguous()).long()
    assert int(want.abs().max()) < 256 and int(sum0.max()) > 1_000_000
    assert torch.equal(y.long(), want)


@pytest.mark.parametrize("M,K,N", [(384, 16384, 2048), (358, 9088, 1024), (1664, 24576, 512)])
def test_a_workspace_without_partial_sums(M, K, N):
    """Grids whose split K wants partial sums, with a workspace that holds the codes and scales only (that
    of a shape on the k groups): served without them, the same output; less is refused."""
    from paper_2609_24433_amd import fq
    flush(f"no partial sums M={M} K={K} N={N}")
    x = synth.activations(M, K, seed=M, outlier_frac=0.01, outlier_scale=30.0).to(DEV)
    wc, sw = fq.quantize_weights(torch.from_numpy(synth.weights(N, K, seed=N)).to(DEV), 128, 4)
    wp = fq.pack_weights(wc, 4)
    least = (M * K // 2 + 255) // 256 * 256 + (M * 4 + 255) // 256 * 256
    full = fq.linear_workspace_bytes(M, N, K, 4)
    assert full > least
    ys = []
    for size in (full, full - 256, least):
        room = torch.full((size + 4096,), 7, dtype=torch.uint8, device=DEV)
        ys.append(fq.linear(x, wp, sw, N, 128, 4, ws=room[:size]))
        torch.cuda.synchronize()
        assert bool((room[size:] == 7).all())  # nothing past the workspace
    assert torch.equal(ys[0], ys[1]) and torch.equal(ys[0], ys[2])
    with pytest.raises(fq.FQError) as e:
        fq.linear(x, wp, sw, N, 128, 4, ws=torch.empty((least - 256,), dtype=torch.uint8, device=DEV))
    assert e.value.status == 5 and str(full) in str(e.value)
