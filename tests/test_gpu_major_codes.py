"""The k-major codes that the fused INT4 projection's prologue writes for the k-group and the
wide-tile GEMM, against the canonical codes of the two separate entry points: the outputs are equal
bit for bit."""
import pytest
import torch

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
