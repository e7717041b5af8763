"""GPTQ kernels at the edges of their blocks: factors whose 64-wide block count is no power of two
(the last merge of a level is narrower), second moments of token counts around the groups of 32,
sweeps of odd row counts, and a diagonal outside the range of the sweep's reciprocal quotient."""
import numpy as np
import pytest
import torch

from paper_2609_24433_amd import synth
from tests.gpu_util import DEV, flush

pytestmark = pytest.mark.gpu


def fq():
    from paper_2609_24433_amd import fq as _fq
    return _fq


@pytest.mark.parametrize("K,T", [(128, 1), (384, 31), (640, 33), (896, 127), (1152, 129)])
def test_second_moment_and_factor(K, T):
    f = fq()
    flush(f"gptq factor K={K} T={T}")
    z = synth.activations(T, K, seed=K + T, outlier_frac=0.01, outlier_scale=30.0).float()
    g = f.gptq_hessian(z.to(DEV))
    want = z.double().numpy().T @ z.double().numpy()
    mag = np.abs(z.double().numpy()).T @ np.abs(z.double().numpy())
    torch.cuda.synchronize()
    # T products in fp64, in any order, twice (numpy's and the kernel's)
    assert np.all(np.abs(g.cpu().numpy() - want) <= 2 * T * 2.0 ** -53 * mag)
    g2 = f.gptq_hessian(z.to(DEV), g.clone(), accumulate=True)
    assert torch.equal(g2, 2 * g) and torch.equal(g, g.t().contiguous())
    u = f.gptq_factor(g, 0.01).cpu().numpy()
    h = want + 0.01 * np.mean(np.diag(want)) * np.eye(K)
    ref = np.linalg.cholesky(np.linalg.inv(h)).T
    assert np.array_equal(u, np.triu(u))
    assert np.abs(u - ref).max() <= 1e-9 * np.abs(ref).max()


@pytest.mark.parametrize("N", [1, 7, 9])
@pytest.mark.parametrize("shift", [-500, 500])
def test_sweep_of_a_scaled_factor(N, shift):
    """A factor times a power of two divides the errors by it and multiplies them back in the
    updates, so the codes stay; at 2^+-500 the quotient is an ordinary division."""
    f = fq()
    K, b = 256, 64
    z = synth.activations(300, K, seed=1, outlier_frac=0.01, outlier_scale=30.0).float().to(DEV)
    u = f.gptq_factor(f.gptq_hessian(z), 0.01)
    w = f.transform(torch.from_numpy(synth.weights(N, K, seed=2)).to(DEV), b)
    codes, scale = f.gptq_sweep(w, u, b, 4)
    codes2, scale2 = f.gptq_sweep(w, u * 2.0 ** shift, b, 4)
    torch.cuda.synchronize()
    assert torch.equal(codes, codes2) and torch.equal(scale, scale2)
    assert bool((codes != f.quantize_weights(torch.from_numpy(synth.weights(N, K, seed=2)).to(DEV), b, 4)[0]).any())
