"""The composite rotation on the fp32 matrix instruction (blocks of 16 channels and more) at the
edges of its row tiles: one row, the last row of a tile and the first of the next, grids on both
sides of the 32-row rule, and workgroups that walk over several tiles with a partial last one.

Bar: codes and scales bit-exact against the oracle's ascending fma chain.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_24433_amd import synth
from tests.gpu_util import DEV, canonical_codes, flush

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,b,bits,weights", [
    (1, 128, 128, 4, False), (15, 256, 16, 8, False), (17, 384, 64, 4, False), (31, 640, 32, 8, False),
    (384, 4096, 64, 4, False), (385, 4096, 64, 4, False),  # 384 tiles of 32 rows, and 416
    (2113, 768, 16, 8, False), (2113, 768, 128, 4, True),  # 402 tiles, one per workgroup; the last of one row
    (1041, 4096, 32, 4, False), (1041, 4096, 128, 8, True),  # 33 row tiles over 16 workgroups
])
def test_matrix_rotation_edges(M, K, b, bits, weights):
    flush(f"rotation edges M={M} K={K} b={b} bits={bits} weights={weights}")
    from paper_2609_24433_amd import fq
    perm, blocks = synth.permutation(K, seed=K + b), synth.orthogonal_blocks(K // b, b, seed=b + 3)
    pre, post = synth.channel_vector(K, seed=1, low=0.25, high=4.0), synth.channel_vector(K, seed=2, low=0.5, high=2.0)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (perm, blocks, pre, post)]
    if weights:
        w = np.random.default_rng(M).standard_normal((M, K)).astype(np.float32)
        codes, scale = fq.quantize_weights_rotated(torch.from_numpy(w).to(DEV), dev[0], dev[1], b, bits, dev[2], dev[3])
        c_ref, s_ref = oracle.quantize_weights_rotated(w, perm, blocks, b, bits, pre, post)
        np.testing.assert_array_equal(codes.cpu().numpy(), c_ref)
    else:
        x = synth.activations(M, K, seed=M + K, outlier_frac=0.01, outlier_scale=30.0)
        codes, scale = fq.rotate_quant(x.to(DEV), dev[0], dev[1], b, bits, 1.0, dev[2], dev[3])
        c_ref, s_ref = oracle.rotate_quant(x, perm, blocks, b, bits, 1.0, pre, post)
        np.testing.assert_array_equal(codes.cpu().numpy(), canonical_codes(c_ref, bits))
    np.testing.assert_array_equal(scale.cpu().numpy(), s_ref)
