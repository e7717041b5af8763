"""The composite rotation of blocks of 1 to 8 channels with four rows per thread (grids of at least 256
workgroups) and with one, at the edges of a workgroup's rows.

Bar: codes and scales bit-exact against the oracle's ascending fma chain.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_24433_amd import synth
from tests.gpu_util import DEV, canonical_codes, flush

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,b", [
    (1, 256, 1), (1025, 256, 1), (3, 512, 2), (1023, 512, 2), (1, 1024, 4), (1024, 1024, 4), (1025, 1024, 4),
    (511, 2048, 8), (513, 2048, 8),  # four rows per thread: 1024 (512 at b = 8) rows a workgroup
    (255, 128, 1), (257, 128, 2), (257, 256, 4), (129, 1024, 8),  # one: 256 (128) rows
])
@pytest.mark.parametrize("bits", [4, 8])
def test_small_blocks(M, K, b, bits):
    flush(f"rotation of small blocks M={M} K={K} b={b} bits={bits}")
    from paper_2609_24433_amd import fq
    x = synth.activations(M, K, seed=M + K, outlier_frac=0.01, outlier_scale=30.0)
    perm, blocks = synth.permutation(K, seed=K + b), synth.orthogonal_blocks(K // b, b, seed=b + 3)
    pre, post = synth.channel_vector(K, seed=1, low=0.25, high=4.0), synth.channel_vector(K, seed=2, low=0.5, high=2.0)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (perm, blocks, pre, post)]
    codes, scale = fq.rotate_quant(x.to(DEV), dev[0], dev[1], b, bits, 1.0, dev[2], dev[3])
    c_ref, s_ref = oracle.rotate_quant(x, perm, blocks, b, bits, 1.0, pre, post)
    np.testing.assert_array_equal(codes.cpu().numpy(), canonical_codes(c_ref, bits))
    np.testing.assert_array_equal(scale.cpu().numpy(), s_ref)
