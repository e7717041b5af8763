"""The GPTQ sweep of more weight rows than one launch of its product update covers (65535 tiles of 32
rows).  Rows are independent: the codes and scales of the rows around that line, and of the last
ones, are those of a sweep of these rows alone.  Rows of zeros and rows with an infinite maximum."""
import pytest
import torch

from paper_2609_24433_amd import synth
from tests.gpu_util import DEV, flush

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [65535 * 32, 65535 * 32 + 1, 65535 * 32 + 77])
def test_sweep_past_one_launch(N):
    from paper_2609_24433_amd import fq
    K, b = 256, 64
    flush(f"gptq sweep N={N} K={K}")
    z = synth.activations(300, K, seed=1, outlier_frac=0.01, outlier_scale=30.0).float().to(DEV)
    u = fq.gptq_factor(fq.gptq_hessian(z), 0.01)
    w = torch.randn((N, K), generator=torch.Generator(device=DEV).manual_seed(N), device=DEV)
    codes, scale = fq.gptq_sweep(w, u, b, 4)
    rows = torch.cat([torch.arange(0, 3), torch.arange(65535 * 32 - 3, N)]).to(DEV)
    codes2, scale2 = fq.gptq_sweep(w[rows].contiguous(), u, b, 4)
    torch.cuda.synchronize()
    assert torch.equal(codes[rows], codes2) and torch.equal(scale[rows], scale2)


@pytest.mark.parametrize("bits", [4, 8])
def test_rows_without_a_step(bits):
    """A row of zeros and rows with an infinite weight (their 1 / step is 0) have codes 0, and leave the
    other rows as they are."""
    from paper_2609_24433_amd import fq
    K, N, b = 384, 11, 64
    flush(f"gptq sweep of rows without a step bits={bits}")
    z = synth.activations(300, K, seed=1, outlier_frac=0.01, outlier_scale=30.0).float().to(DEV)
    u = fq.gptq_factor(fq.gptq_hessian(z), 0.01)
    w = torch.randn((N, K), generator=torch.Generator(device=DEV).manual_seed(N), device=DEV)
    codes, scale = fq.gptq_sweep(w, u, b, bits)
    bad = w.clone()
    bad[2] = 0.0
    bad[3, 0] = bad[4, 200] = float("inf")
    bad[7, 383] = -float("inf")
    codes2, scale2 = fq.gptq_sweep(bad, u, b, bits)
    torch.cuda.synchronize()
    odd = [2, 3, 4, 7]
    rest = [i for i in range(N) if i not in odd]
    assert not codes2[odd].any() and float(scale2[2]) == 0.0 and bool(torch.isinf(scale2[[3, 4, 7]]).all())
    assert torch.equal(codes2[rest], codes[rest]) and torch.equal(scale2[rest], scale[rest])
