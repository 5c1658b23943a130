"""Rows of dY and of W in one launch: the bits of the two tensors quantized apart, at row counts that leave a workgroup's part empty or
divided between the two, with the column maxima beside (bf16, one call) and without, for every number of columns' own kernel."""
import pytest
import torch

from paper_2501_17116_amd import binding as b

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,K,N", [(32, 32, 32), (96, 40, 1056), (32, 1056, 2080), (1056, 72, 4128), (64, 64, 8224), (32, 72, 12320), (32, 64, 16416)])
def test_the_bits_of_both_apart(M, K, N, dtype):
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    dY = (torch.randn(M, N, generator=g, device="cuda") * 0.01).to(dtype)
    W = (torch.randn(K, N, generator=g, device="cuda") * torch.rand(K, 1, generator=g, device="cuda")).to(dtype)
    qY, gY = b.fp4_quantize(dY, b.FP4_AXIS_ROW)
    qW, gW = b.fp4_quantize(W, b.FP4_AXIS_ROW)
    want = b.fp4_gemm(qY, gY, qW, gW, out_dtype=dtype)
    assert torch.equal(b.fp4_linear_bwd_dgrad(dY, W), want)
    if K % 32 == 0:
        A = torch.randn(M, K, generator=g, device="cuda").to(dtype)
        _, ctx = b.fp4_linear_fwd(A, W, 1.0)
        dA, dW = b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0)
        assert torch.equal(dA, want)
        assert torch.equal(dW, b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0))
