"""What small layers launch beside each other: the first digit pass over A beside the codes of W, the residual's transposition beside dY's
rows and beside the weight gradient's codes.  Each against the same work launched by itself, at the smallest sizes, at columns and rows that
are no whole tile, on either side of 4096 columns (the count of the entries) and of what finds room on the chip at once; bits are the same."""
import pytest
import torch

from paper_2501_17116_amd import binding as b

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,K,N", [(32, 32, 32), (64, 64, 8224), (96, 4096, 96), (96, 4128, 64), (288, 8192, 160), (1056, 1376, 2080), (2048, 512, 2080),
                                   (2304, 2048, 2080), (4128, 4096, 288)])
def test_same_as_by_themselves(M, K, N, dtype):
    alpha = 0.97
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    A = torch.randn(M, K, generator=g, device="cuda")
    A[:, K // 2] *= 20
    A, W = A.to(dtype), (torch.randn(K, N, generator=g, device="cuda") * 0.02).to(dtype)
    dY = (torch.randn(M, N, generator=g, device="cuda") * 0.01).to(dtype)
    Y, ctx = b.fp4_linear_fwd(A, W, alpha)
    want = b.occ_clamp_residual(A, alpha)
    n = int(want["nnz"])
    assert torch.equal(ctx.nnz, want["nnz"]) and torch.equal(ctx.thresholds, want["thresholds"]) and torch.equal(ctx.row_ptr, want["row_ptr"])
    assert torch.equal(ctx.col_idx[:n], want["col_idx"][:n]) and torch.equal(ctx.val[:n], want["val"][:n])
    wq = b.fp4_prepare_weights(W)
    assert torch.equal(ctx.gamma_W, wq.gamma_W)
    assert torch.equal(Y, b.fp4_linear_fwd_cached(A, W, wq, alpha)[0])
    dA, dW = b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0)
    assert torch.equal(dA, b.fp4_linear_bwd_dgrad(dY, W))
    assert torch.equal(dW, b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0))
