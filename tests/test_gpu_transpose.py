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


@pytest.mark.parametrize("M,K", [(1, 32), (33, 64), (64, 4096), (96, 4128), (200, 8192), (65, 8224), (300, 16384), (4096, 96), (4128, 96), (9000, 32),
                                 (64, 16416)])
def test_every_entry_in_its_place(M, K):
    """By each way of finding the places, at a last block that is whole or not, columns and rows that are empty or full."""
    g = torch.Generator(device="cuda").manual_seed(M + K)
    mask = torch.rand(M, K, generator=g, device="cuda") < 0.05
    mask[:, :8] = False
    mask[M // 2] = False
    if M > 1:
        mask[:, K // 3] = True
        mask[M // 3] = True
        mask[M - 1, 8:] |= torch.rand(K - 8, generator=g, device="cuda") < 0.3
    mask &= torch.cumsum(mask.flatten(), 0).view(M, K) <= b.occ_capacity(M, K, 0.9)
    ptr = torch.zeros(M + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(mask.sum(1), 0, out=ptr[1:])
    if int(ptr[-1]) == 0:
        return
    S = torch.randn(M, K, generator=g, device="cuda")
    col, val = mask.nonzero()[:, 1].int().contiguous(), S[mask].contiguous()
    want_ptr = torch.zeros(K + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(mask.sum(0), 0, out=want_ptr[1:])
    want_idx, want_val = mask.t().nonzero()[:, 1].int(), S.t()[mask.t()]
    for positions in ((0, 1, 2, 3) if K <= 16384 else (0,)):
        t_ptr, t_idx, t_val = b.fp4_residual_transpose(ptr, col, val, ptr[-1:].clone(), K, positions)
        assert torch.equal(t_ptr, want_ptr), positions
        assert torch.equal(t_idx, want_idx), positions
        assert torch.equal(t_val, want_val), positions
