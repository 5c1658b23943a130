"""The FP4 GEMM's small-tile kernel at the edges of its tiles, and products on either side of the lines between it and the
128 x 128 tiles: against the exact integer product (raw accumulators) and, scaled, bit for bit against a problem large enough
for the 256 x 256 tiles that holds the same rows and columns."""
import pytest
import torch

pytestmark = pytest.mark.gpu

GRID = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6])


def _values(codes):
    return GRID[torch.stack([codes & 15, codes >> 4], -1).reshape(codes.shape[0], -1).long()]


@pytest.mark.parametrize("P,Q,K", [(1, 8, 32), (63, 72, 96), (64, 64, 256), (65, 136, 288), (512, 2048, 64), (520, 2056, 160),
                                   (1000, 1024, 2080), (1024, 1024, 512)])
def test_small_tiles(P, Q, K):
    from paper_2501_17116_amd import binding as b
    g = torch.Generator().manual_seed(P + Q + K)
    L = torch.randint(0, 256, (P, K // 2), generator=g, dtype=torch.uint8)
    R = torch.randint(0, 256, (Q, K // 2), generator=g, dtype=torch.uint8)
    raw = b.fp4_gemm(L.cuda(), None, R.cuda(), None).cpu()
    assert torch.equal(raw.double(), _values(L).double() @ _values(R).double().t())
    gl, gr = torch.rand(P, generator=g) + 0.5, torch.rand(Q, generator=g) + 0.5
    Pb, Qb = 3072, 3072   # 144 tiles of 256 x 256
    Lb, Rb = torch.zeros(Pb, K // 2, dtype=torch.uint8), torch.zeros(Qb, K // 2, dtype=torch.uint8)
    Lb[:P], Rb[:Q] = L, R
    glb, grb = torch.ones(Pb), torch.ones(Qb)
    glb[:P], grb[:Q] = gl, gr
    for dt in (torch.float32, torch.bfloat16):
        small = b.fp4_gemm(L.cuda(), gl.cuda(), R.cuda(), gr.cuda(), out_dtype=dt)
        big = b.fp4_gemm(Lb.cuda(), glb.cuda(), Rb.cuda(), grb.cuda(), out_dtype=dt)
        assert torch.equal(small, big[:P, :Q])


@pytest.mark.parametrize("M,K,N", [(3072, 2048, 2048), (3104, 2048, 2048), (6144, 2048, 1024), (6176, 2048, 1024), (32, 64, 72)])
def test_fp32_factor(M, K, N):
    """The weight gradient with fp32 masters, on 128 x 128 tiles in rounds and part rounds and on one of 64 x 64, against its
    parts called one by one (the factor as a pass of its own): the product is the same to the last bit, the factor one
    rounding of fp32 in either."""
    from paper_2501_17116_amd import binding as b
    torch.manual_seed(M + N)
    A, W, dY = torch.randn(M, K, device="cuda"), torch.randn(K, N, device="cuda") * 0.02, torch.randn(M, N, device="cuda")
    _, ctx = b.fp4_linear_fwd(A, W, 1.0)
    got = b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0)
    qA, gA = b.fp4_quantize(A, b.FP4_AXIS_COL)
    qY, gY = b.fp4_quantize(dY, b.FP4_AXIS_COL)
    ref = b.fp4_dge_apply(b.fp4_gemm(qA, gA, qY, gY), W, ctx.gamma_W, 5.0, 3.0)
    assert torch.all((got - ref).abs() <= 2.0 ** -22 * ref.abs())


@pytest.mark.parametrize("P,Q", [(65, 72), (4096, 4104)])
def test_an_empty_contraction(P, Q):
    """No codes at all, and no operands: the addend alone."""
    from paper_2501_17116_amd import binding as b
    addend = torch.randn(P, Q, device="cuda")
    out = torch.full((P, Q), float("nan"), device="cuda")
    assert b.lib().fp4_gemm(None, None, None, None, P, Q, 0, b._ptr(addend), b._ptr(out), b.FP4_F32, Q, b._stream()) == 0
    assert torch.equal(out, addend)


@pytest.mark.parametrize("P,Q,K,tile", [(512, 2048, 1280, 64), (512, 2048, 1536, 128), (520, 2048, 256, 64), (520, 2048, 512, 128),
                                        (520, 2056, 1056, 64), (520, 2056, 1120, 128), (1032, 2056, 416, 64), (1032, 2056, 480, 128),
                                        (192, 4136, 4384, 64), (192, 4136, 4416, 128), (776, 1032, 1120, 64), (776, 1032, 1536, 128)])
def test_either_side_of_the_lines_between_the_tilings(P, Q, K, tile):
    """Under scales of any value: the rows of a problem that the 256 x 256 tiles take, to the last bit."""
    from paper_2501_17116_amd import binding as b
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus != 256 or b.fp4_gemm_tiling(P, Q, K)[0] == tile
    g = torch.Generator(device="cuda").manual_seed(P + Q + K)
    Pb, Qb = 4608, 4352   # 306 tiles
    L = torch.randint(0, 256, (Pb, K // 2), generator=g, dtype=torch.uint8, device="cuda")
    R = torch.randint(0, 256, (Qb, K // 2), generator=g, dtype=torch.uint8, device="cuda")
    gl, gr = torch.rand(Pb, generator=g, device="cuda") + 0.5, torch.rand(Qb, generator=g, device="cuda") + 0.5
    addend = torch.randn(Pb, Qb, generator=g, device="cuda")
    for dt in (torch.float32, torch.bfloat16):
        one = b.fp4_gemm(L[:P], gl[:P], R[:Q], gr[:Q], out_dtype=dt, addend=addend[:P, :Q].contiguous())
        big = b.fp4_gemm(L, gl, R, gr, out_dtype=dt, addend=addend)
        assert torch.equal(one, big[:P, :Q])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,K,N", [(3072, 512, 2048), (3328, 512, 2048), (768, 520, 2048), (1024, 520, 2048), (256, 1032, 2048), (512, 1032, 2048),
                                   (6016, 1024, 832), (8480, 512, 512), (8480, 264, 136), (3328, 136, 264),   # 32 x 32, three of them
                                   (8160, 1024, 1024), (8224, 1024, 1024), (8224, 904, 1032), (3328, 904, 1032), (1312, 520, 2048), (2400, 1280, 1280), (1184, 1032, 2048),
                                   (1376, 1032, 2048), (1408, 1032, 2048), (640, 672, 5496), (672, 672, 5496)])
def test_factor_on_either_side_of_the_lines(M, K, N, dtype):
    """The weight gradient against its parts called one by one: the product is the same to the last bit, the factor one
    rounding of fp32 in either."""
    from paper_2501_17116_amd import binding as b
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert (b.fp4_gemm_tiling(K, N, M, True, dtype == torch.bfloat16)[0] == 32) == (K * N <= 512 * 1024 and M >= 256)
    torch.manual_seed(M + N)
    A, W, dY = (t.to(dtype) for t in (torch.randn(M, K, device="cuda"), torch.randn(K, N, device="cuda") * 0.02, torch.randn(M, N, device="cuda")))
    _, ctx = b.fp4_linear_fwd(A[:, :K // 32 * 32].contiguous(), W[:K // 32 * 32].contiguous(), 1.0)
    got = b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0)
    qA, gA = b.fp4_quantize(A, b.FP4_AXIS_COL)
    qY, gY = b.fp4_quantize(dY, b.FP4_AXIS_COL)
    ref = b.fp4_dge_apply(b.fp4_gemm(qA, gA, qY, gY), W, ctx.gamma_W, 5.0, 3.0)
    assert torch.all((got - ref).abs() <= 2.0 ** -22 * ref.abs())
