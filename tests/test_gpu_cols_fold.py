"""Column-wise quantization, whose tiles form the scales from partial maxima: the codes and scales are those of the transposed
tensor quantized by rows, bit for bit, whatever the number of row blocks and however the last tiles are cut."""
import pytest
import torch

from paper_2501_17116_amd import binding as b

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,cols", [(8, 8), (40, 56), (264, 72), (480, 2080), (2080, 72), (4128, 1032), (16416, 520), (131072, 512)])
def test_columns_are_the_transposed_tensors_rows(rows, cols, dtype):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = torch.randn(rows, cols, generator=g, device="cuda").to(dtype)
    x[:, 1::3] *= 30.0
    codes, gamma = b.fp4_quantize(x, b.FP4_AXIS_COL)
    want, want_gamma = b.fp4_quantize(x.t().contiguous(), b.FP4_AXIS_ROW)
    assert torch.equal(gamma, want_gamma)
    assert torch.equal(codes, want)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,K,N", [(32, 32, 64), (1056, 1376, 2080), (8192, 512, 4096), (4096, 64, 13824)])
def test_both_gradients_in_one_call_or_two(M, K, N, dtype):
    """The operands of the weight gradient share launches; with dY's maxima from the dual-axis pass (bf16, one call) or without."""
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    A, W = (torch.randn(*s, generator=g, device="cuda").to(dtype) for s in ((M, K), (K, N)))
    dY = (torch.randn(M, N, generator=g, device="cuda") * 0.01).to(dtype)
    _, ctx = b.fp4_linear_fwd(A, W, 0.99)
    dA, dW = b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0)
    assert torch.equal(dA, b.fp4_linear_bwd_dgrad(dY, W))
    assert torch.equal(dW, b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0))
