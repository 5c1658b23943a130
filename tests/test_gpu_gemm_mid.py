"""The FP4 GEMM's 128 x 128 tiles at the edges of tiles, ring and dispatch, and its 256 x 256 tiles on contractions that end
inside a K step: against the exact integer product (raw accumulators; every sum is a multiple of 1/4 below 2^22)
and, scaled, against the definition's fp32 operations on it, to the last bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu

GRID = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6])


def _values(codes):
    return GRID[torch.stack([codes & 15, codes >> 4], -1).reshape(codes.shape[0], -1).long()]


@pytest.mark.parametrize("P,Q,K", [(1, 8, 1056), (127, 136, 1280), (128, 128, 1312), (129, 1000, 2048), (2048, 2048, 32),   # 64 x 64 and 32 x 32
                                   (2049, 2056, 288), (2176, 3840, 1024), (4096, 2048, 544),      # 128 x 128; 512 of them
                                   (4096, 2056, 544), (2816, 3080, 32), (2816, 3072, 288), (4352, 4096, 992),   # 256 x 256
                                   (4104, 4104, 32), (4224, 4232, 544), (4352, 4352, 1024), (5120, 4096, 160)])   # and a last round in quarters
def test_products(P, Q, K):
    from paper_2501_17116_amd import binding as b
    g = torch.Generator().manual_seed(P + Q + K)
    L = torch.randint(0, 256, (P, K // 2), generator=g, dtype=torch.uint8)
    R = torch.randint(0, 256, (Q, K // 2), generator=g, dtype=torch.uint8)
    exact = _values(L).cuda() @ _values(R).cuda().t()   # exact in fp32: no partial sum needs more than 24 bits
    L, R = L.cuda(), R.cuda()
    assert torch.equal(b.fp4_gemm(L, None, R, None), exact)
    # powers of two: reciprocals and products without rounding, whatever the order
    gl, gr = (torch.exp2(torch.randint(-3, 4, (n,), generator=g).float()).cuda() for n in (P, Q))
    addend = torch.randn(P, Q, generator=g).cuda()
    scaled = exact / gl[:, None] / gr
    assert torch.equal(b.fp4_gemm(L, gl, R, gr, out_dtype=torch.bfloat16), scaled.bfloat16())
    assert torch.equal(b.fp4_gemm(L, gl, R, gr, addend=addend), scaled + addend)


@pytest.mark.parametrize("P,Q,K", [(33, 12296, 1536), (127, 6152, 1792), (128, 6272, 6176), (129, 5000, 6208), (127, 6280, 6304), (1, 24584, 1536)])
def test_edges_of_a_tile(P, Q, K):
    """Contractions long enough for 128 x 128 tiles, at the fewest rows and outputs just past what 32 x 32 tiles take."""
    from paper_2501_17116_amd import binding as b
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert b.fp4_gemm_tiling(P, Q, K)[0] == 128
    test_products(P, Q, K)


@pytest.mark.parametrize("P,Q,K", [(4352, 4352, 544), (4104, 4360, 1024), (4224, 4360, 288), (2056, 8456, 96)])
def test_a_last_round_in_quarters_gives_the_same_bits(P, Q, K):
    """Under scales of any value: the rows of a problem twice as high, whose 256 x 256 tiles are all left whole."""
    from paper_2501_17116_amd import binding as b
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert b.fp4_gemm_tiling(P, Q, K)[:2] > (256, 0) and b.fp4_gemm_tiling(2 * P, Q, K)[:2] == (256, 0)
    g = torch.Generator(device="cuda").manual_seed(P + Q + K)
    L = torch.randint(0, 256, (2 * P, K // 2), generator=g, dtype=torch.uint8, device="cuda")
    R = torch.randint(0, 256, (Q, K // 2), generator=g, dtype=torch.uint8, device="cuda")
    gl, gr = torch.rand(2 * P, generator=g, device="cuda") + 0.5, torch.rand(Q, generator=g, device="cuda") + 0.5
    addend = torch.randn(2 * P, Q, generator=g, device="cuda")
    for dt in (torch.float32, torch.bfloat16):
        for ad in (None, addend):
            cut = b.fp4_gemm(L[:P], gl[:P], R, gr, out_dtype=dt, addend=None if ad is None else ad[:P])
            assert torch.equal(cut, b.fp4_gemm(L, gl, R, gr, out_dtype=dt, addend=ad)[:P])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,K,N", [(96, 1280, 1288), (1056, 1376, 2080), (2080, 1056, 2056), (2048, 2048, 2048), (1056, 3104, 3080), (544, 4128, 4112)])
def test_weight_gradient_with_the_factor(M, K, N, dtype):
    """Against its parts called one by one (the factor as a pass of its own): the same product to the last bit, the factor one
    rounding of fp32 in either."""
    from paper_2501_17116_amd import binding as b
    torch.manual_seed(M + N)
    A, W, dY = (t.to(dtype) for t in (torch.randn(M, K, device="cuda"), torch.randn(K, N, device="cuda") * 0.02, torch.randn(M, N, device="cuda")))
    _, ctx = b.fp4_linear_fwd(A, W, 1.0)
    got = b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0)
    qA, gA = b.fp4_quantize(A, b.FP4_AXIS_COL)
    qY, gY = b.fp4_quantize(dY, b.FP4_AXIS_COL)
    ref = b.fp4_dge_apply(b.fp4_gemm(qA, gA, qY, gY), W, ctx.gamma_W, 5.0, 3.0)
    assert torch.all((got - ref).abs() <= 2.0 ** -22 * ref.abs())
