"""The residual's transpose inside the weight gradient, at the sizes where its positions come from another place: counts of
all row blocks in the filling workgroup (up to 64 Ki of them), pass 2's scan beyond that, blocks of 32 rows above 8192 columns."""
import numpy as np
import pytest
import torch

from oracle import fp4_oracle as o
from paper_2501_17116_amd import binding as b

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K", [(32, 64), (96, 4128), (1024, 4096), (1056, 4096), (512, 8192), (544, 8192), (96, 8224), (224, 8224), (256, 8224), (96, 16384)])
def test_weight_gradient_of_a_residual(M, K):
    N, alpha, k, cap = 32, 0.97, 5.0, 3.0
    g = torch.Generator().manual_seed(M + K)
    A = torch.randn(M, K, generator=g)
    A[:, torch.randperm(K, generator=g)[:3]] *= 20.0
    W, dY = torch.randn(K, N, generator=g) * 0.02, torch.randn(M, N, generator=g) * 0.01
    _, ctx = b.fp4_linear_fwd(A.cuda(), W.cuda(), alpha)
    got = b.fp4_linear_bwd_wgrad(A.cuda(), dY.cuda(), W.cuda(), ctx, k, cap).cpu().numpy().astype(np.float64)
    ref = o.fp4_linear_bwd_wgrad(A.numpy(), dY.numpy(), W.numpy(), alpha, k, cap).astype(np.float64)
    # fp32 sums of up to M terms, and the factor's own error (1e-3 next to its pole): the bar of the layer's other fp32 tests
    assert np.all(np.abs(got - ref) <= 1e-3 * np.abs(ref) + 2e-6 * np.abs(ref).max())
