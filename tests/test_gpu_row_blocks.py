"""Column scales where the number of rows a workgroup folds changes with the tensor's size (partial maxima of 4 to 32
rows in the dual-axis pass, 32 to 128 in the column pass): bit for bit those of torch's column maxima, codes those of an
independent rounding under them, and the dual-axis pass the same as the separate ones."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _codes(x):
    """E2M1 codes of x: nearest, midpoints up, saturating; no negative zero."""
    grid = torch.tensor([-6, -4, -3, -2, -1.5, -1, -.5, 0, .5, 1, 1.5, 2, 3, 4, 6], device=x.device)
    code = torch.tensor([15, 14, 13, 12, 11, 10, 9, 0, 1, 2, 3, 4, 5, 6, 7], dtype=torch.uint8, device=x.device)
    return code[torch.bucketize(x, (grid[1:] + grid[:-1]) / 2, right=True)]


@pytest.mark.parametrize("M,K,N", [(32, 32, 32), (64, 8, 8224), (1056, 64, 2080), (4096, 32, 96), (4128, 40, 8224), (8192, 32, 32),
                                   (16384, 32, 64), (32768, 8, 32), (4128, 8, 512), (8192, 8, 512), (8224, 8, 520), (16416, 8, 512)])
def test_column_scales(M, K, N):
    from paper_2501_17116_amd import binding as b
    torch.manual_seed(M + N)
    dY = (torch.randn(M, N, device="cuda") * torch.exp(torch.randn(1, N, device="cuda"))).bfloat16()
    codes, gamma = b.fp4_quantize(dY, b.FP4_AXIS_COL)
    assert torch.equal(gamma, (6.0 / dY.float().abs().amax(0).double()).float())
    c = _codes(dY.float() * gamma).t()
    assert torch.equal(codes, c[:, 0::2] | c[:, 1::2] << 4)
    if K % 32 == 0:   # the dual-axis pass of the one-call backward against the separate calls
        A, W = torch.randn(M, K, device="cuda").bfloat16(), torch.randn(K, N, device="cuda").bfloat16()
        Y, ctx = b.fp4_linear_fwd(A, W, 0.99)
        dA, dW = b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0)
        assert torch.equal(dA, b.fp4_linear_bwd_dgrad(dY, W))
        assert torch.equal(dW, b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0))
