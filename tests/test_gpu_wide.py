"""The wide-tile GEMMs of both widths and the INT4 k groups on the FP6 matrix cores at the edges of
their tiles and plans.  Through the library's entry points: the fused projection (its prologue
writing k-major codes) equal bit for bit to the prologue and the GEMM on
canonical codes, and the GEMM's accumulators equal to numpy's integer product on rows at the tile
boundaries."""
import numpy as np
import pytest
import torch

from paper_2609_24433_amd import synth
from tests.gpu_util import DEV, flush

pytestmark = pytest.mark.gpu


def fq():
    from paper_2609_24433_amd import fq as _fq
    return _fq


# (M, K, N): wide tiles need more than 256 tiles of 128 x 128 (INT4 3 k steps), k groups K >= 4096 and
# at most 256 tiles of 128 x 64 (up to 256 of 128 x 128 from K = 8192 on, but more than 64).  Ragged
# last row blocks (M % 32, M % 256), ragged last column tiles (N % 128, N % 64), k steps that are no
# multiple of 4 or 3, one k step.
SHAPES = [(129, 128, 16400), (257, 384, 11040), (1000, 1152, 4240), (2049, 640, 2064), (4095, 1664, 1040),
          (65, 4096, 1040), (97, 4224, 2064), (333, 6272, 1552), (513, 8320, 3088), (801, 16512, 1040),
          # grids of up to 64 tiles of 128 x 128 from K = 8192 on: the LDS-ring kernel
          (358, 9088, 816), (358, 8192, 1024)]


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_fused_equals_split(M, K, N, bits):
    f = fq()
    flush(f"wide M={M} K={K} N={N} bits={bits}")
    b = 128
    x = synth.activations(M, K, seed=M + K, outlier_frac=0.01, outlier_scale=30.0).to(DEV)
    w = torch.from_numpy(synth.weights(N, K, seed=N)).to(DEV)
    bias = torch.from_numpy(synth.random_scales(N, seed=3, low=-0.1, high=0.1)).to(DEV)
    wc, sw = f.quantize_weights(w, b, bits)
    wp = f.pack_weights(wc, bits)
    ld = N + 8
    out = torch.full((M, ld), 7.0, dtype=torch.bfloat16, device=DEV)  # columns past N stay as they are
    f.linear(x, wp, sw, N, b, bits, bias=bias, out=out[:, :N])
    codes, delta = f.fwht_quant(x, b, bits)
    y, acc = f.gemm(codes, delta, wp, sw, N, K, bits, bias, want_acc=True)
    torch.cuda.synchronize()
    assert torch.equal(out[:, :N], y)
    assert bool((out[:, N:] == 7.0).all())
    rows = sorted({0, 31, 32, 127, 128, 255, 256, M - 33, M - 1} & set(range(M)))
    c = codes[rows].cpu().numpy()
    if bits == 4:  # channel 2i in the low nibble of byte i, two's complement
        a = ((np.stack([c & 15, c >> 4], axis=2).reshape(len(rows), K).astype(np.int64) ^ 8) - 8)
    else:
        a = c.view(np.int8)
    want = a.astype(np.int64) @ wc.cpu().numpy().astype(np.int64).T
    assert np.array_equal(acc[rows].cpu().numpy().astype(np.int64), want)


@pytest.mark.parametrize("M,N", [(816, 2048), (2064, 2064)])
def test_largest_sums_are_exact(M, N):
    """Every code 7 at K = 32768: the six-bit fields hold 15, their products' fp32 sums reach
    225 * 32768, and the accumulators come out as 49 * 32768 to bf16's rounding (to the last unit:
    test_gpu_major_codes.py, test_long_sums_to_the_last_unit)."""
    f = fq()
    K = 32768
    x = torch.ones((M, K), dtype=torch.bfloat16, device=DEV)
    w = torch.ones((N, K), dtype=torch.float32, device=DEV)
    wc, sw = f.quantize_weights(w, 1, 4)
    y = f.linear(x, f.pack_weights(wc, 4), torch.ones_like(sw), N, 1, 4)
    delta = f.fwht_quant(x, 1, 4)[1]
    want = (torch.full((M, N), 49.0 * K, device=DEV) * delta[:, None]).to(torch.bfloat16)
    torch.cuda.synchronize()
    assert bool((wc == 7).all()) and torch.equal(y, want)

