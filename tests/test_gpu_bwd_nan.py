"""A NaN in dY or W: both gradients in one call, weights cached or not, are bit for bit what the separate calls give, whose row and
column maxima are those of the other elements."""
import pytest
import torch

from paper_2501_17116_amd import binding as b

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("where", ["W", "dY", "both"])
@pytest.mark.parametrize("M,K,N", [(64, 96, 512), (96, 64, 4128), (1280, 64, 2080), (32, 64, 12320)])
def test_one_call_or_two(M, K, N, where, dtype):
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    A = torch.randn(M, K, generator=g, device="cuda").to(dtype)
    W = torch.randn(K, N, generator=g, device="cuda").to(dtype)
    dY = (torch.randn(M, N, generator=g, device="cuda") * 0.01).to(dtype)
    _, ctx = b.fp4_linear_fwd(A, W, 0.99)
    # the largest elements of the NaN's thread: its eight neighbours, and where a thread has more, those 2048 columns on
    for x, r in ((W, 5), (dY, 3)):
        x[r, 16] = 50.0
        x[r, 17 if N < 2048 else 2064] = -60.0
    if where != "dY":
        W[5, 18] = float("nan")
        W[K - 1, N - 1] = -float("nan")
    if where != "W":
        dY[3, 18] = float("nan")
        dY[M - 1, 1::7] = float("nan")
        dY[:, 8] = float("nan")
    wq = b.fp4_prepare_weights(W)
    want_A, want_W = b.fp4_linear_bwd_dgrad(dY, W), b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0)
    for cache in (None, wq):
        dA, dW = b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0, wq=cache)
        assert torch.equal(dA, want_A)
        assert torch.equal(dW.view(torch.int32), want_W.view(torch.int32))
