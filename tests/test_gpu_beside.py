"""What small layers launch beside each other: the first digit pass over A beside the codes of W, the residual's transposition beside dY's
rows and beside the weight gradient's codes.  Each against the same work launched by itself (fp4_linear_fwd_cached, occ_clamp_residual, and for the
weight gradient its parts: fp4_quantize, fp4_residual_transpose, fp4_residual_spmm, fp4_gemm), at the smallest sizes, at columns and rows that
are no whole tile, with one, two and four tiles a workgroup and on the other side of each line (`fill`, `bf16` and `f32`: tiles a workgroup of the
codes beside the transposition's last pass, and beside the digit pass over an A of either type); bits are the same."""
import pytest
import torch

from paper_2501_17116_amd import binding as b

pytestmark = pytest.mark.gpu

SHAPES = [
    # M, K, N, fill, bf16, f32
    (32, 32, 32, 1, 1, 1), (64, 64, 8224, 1, 1, 1), (96, 4096, 96, 1, 1, 1), (96, 4128, 64, 1, 1, 1), (288, 8192, 160, 1, 1, 1),
    (1056, 1376, 2080, 1, 1, 1), (2048, 512, 2080, 1, 1, 1), (2304, 2048, 2080, 2, 1, 2), (4128, 4096, 288, 4, 1, 1),
    (1056, 8192, 2080, 2, 0, 0), (6144, 2048, 2080, 4, 1, 2), (2080, 4128, 2080, 2, 1, 0), (64, 4096, 4128, 1, 0, 4), (32, 4096, 8192, 1, 0, 0),
    (8224, 2048, 2080, 0, 1, 2), (96, 8224, 160, 0, 1, 1),
]


def _inputs(M, K, N, dtype):
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    A = torch.randn(M, K, generator=g, device="cuda")
    A[:, K // 2] *= 20
    return A.to(dtype), (torch.randn(K, N, generator=g, device="cuda") * 0.02).to(dtype), (torch.randn(M, N, generator=g, device="cuda") * 0.01).to(dtype)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("scope", [b.FP4_OCC_TENSOR, b.FP4_OCC_TOKEN])
@pytest.mark.parametrize("M,K,N,fill,bf16,f32", SHAPES)
def test_same_as_by_themselves(M, K, N, fill, bf16, f32, scope, dtype):
    alpha = 0.97
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert b.fp4_transpose_beside(M, K, N) == fill
        assert b.fp4_select_beside(M, K, N, b.FP4_BF16) == bf16 and b.fp4_select_beside(M, K, N, b.FP4_F32) == f32
    A, W, dY = _inputs(M, K, N, dtype)
    Y, ctx = b.fp4_linear_fwd(A, W, alpha, scope=scope)
    want = b.occ_clamp_residual(A, alpha, want_clamped=True, scope=scope)
    n = int(want["nnz"])
    assert torch.equal(ctx.nnz, want["nnz"]) and torch.equal(ctx.thresholds, want["thresholds"]) and torch.equal(ctx.row_ptr, want["row_ptr"])
    assert torch.equal(ctx.col_idx[:n], want["col_idx"][:n]) and torch.equal(ctx.val[:n], want["val"][:n])
    wq = b.fp4_prepare_weights(W)
    assert torch.equal(ctx.gamma_W, wq.gamma_W)
    assert torch.equal(Y, b.fp4_linear_fwd_cached(A, W, wq, alpha, ctx=b.FwdCtx(M, K, N, alpha, scope=scope))[0])
    dA, dW = b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0)
    assert torch.equal(dA, b.fp4_linear_bwd_dgrad(dY, W))
    assert torch.equal(dW, b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0))
    # without the derivative factor, from its parts
    t_ptr, t_idx, t_val = b.fp4_residual_transpose(ctx.row_ptr, ctx.col_idx, ctx.val, ctx.nnz, K)
    R = b.fp4_residual_spmm(t_ptr, t_idx[:max(ctx.capacity, 1)], t_val[:max(ctx.capacity, 1)], M, dY)
    qA, gA = b.fp4_quantize(want["x_clamped"], b.FP4_AXIS_COL)
    qY, gY = b.fp4_quantize(dY, b.FP4_AXIS_COL)
    parts = b.fp4_gemm(qA, gA, qY, gY, addend=R)
    assert torch.equal(b.fp4_linear_bwd(dY, A, W, ctx, 0.0, 0.0)[1], parts)
    assert torch.equal(b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 0.0, 0.0), parts)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,K,N,alpha", [(32, 32, 32, 0.9), (96, 3072, 96, 0.999), (512, 1376, 2080, 0.99), (512, 1376, 2080, 0.97), (96, 1376, 8224, 0.97),
                                         (96, 256, 16416, 0.97), (96, 2048, 11040, 0.99)])
def test_count_beside_the_rows(M, K, N, alpha, dtype):
    """The transposition's first pass beside the rows of narrow and wide dY (one with a row's units in each of the kernel's forms) and W."""
    A, W, dY = _inputs(M, K, N, dtype)
    ctx = b.fp4_linear_fwd(A, W, alpha)[1]
    want = b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0)   # counts in a launch of its own
    assert torch.equal(b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0)[1], want)
    assert torch.equal(b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0, wq=b.fp4_prepare_weights(W))[1], want)
