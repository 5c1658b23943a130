"""Column scales where the number of rows a workgroup folds changes with the tensor's size (partial maxima of 4 to 32
rows in the dual-axis pass, 32 to 128 in the column pass): bit for bit torch's column maxima, codes as fp4_quantize."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(32, 32, 32), (64, 8, 8224), (1056, 64, 2080), (4096, 32, 96), (4128, 40, 8224), (8192, 32, 32),
                                   (16384, 32, 64), (32768, 8, 32)])
def test_column_scales(M, K, N):
    from paper_2501_17116_amd import binding as b
    torch.manual_seed(M + N)
    dY = (torch.randn(M, N, device="cuda") * torch.exp(torch.randn(1, N, device="cuda"))).bfloat16()
    codes, gamma = b.fp4_quantize(dY, b.FP4_AXIS_COL)
    assert torch.equal(gamma, (6.0 / dY.float().abs().amax(0).double()).float())
    if K % 32 == 0:   # the dual-axis pass of the one-call backward against the separate calls
        A, W = torch.randn(M, K, device="cuda").bfloat16(), torch.randn(K, N, device="cuda").bfloat16()
        Y, ctx = b.fp4_linear_fwd(A, W, 0.99)
        dA, dW = b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0)
        assert torch.equal(dA, b.fp4_linear_bwd_dgrad(dY, W))
        assert torch.equal(dW, b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0))
