"""The FP4 GEMM's 32 x 32 tiles, whose waves share a contraction: at the edges of tiles, with fewer K steps than waves, a last step that
overhangs the row, rings of four and of two steps; raw against the exact integer product, scaled bit for bit against a problem that the
256 x 256 tiles take."""
import pytest
import torch

pytestmark = pytest.mark.gpu

GRID = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6])


def _values(codes):
    return GRID[torch.stack([codes & 15, codes >> 4], -1).reshape(codes.shape[0], -1).long()]


@pytest.mark.parametrize("P,Q,K", [(1, 8, 512), (31, 40, 768), (32, 32, 1024), (33, 72, 1120), (64, 64, 1280), (65, 136, 4128), (32, 264, 8192),
                                   (264, 1024, 512), (250, 2040, 1376), (512, 1024, 2560), (512, 1528, 3104)])
def test_against_the_exact_product(P, Q, K):
    from paper_2501_17116_amd import binding as b
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus != 256 or b.fp4_gemm_splits(P, Q, K)
    g = torch.Generator().manual_seed(P + Q + K)
    L = torch.randint(0, 256, (P, K // 2), generator=g, dtype=torch.uint8)
    R = torch.randint(0, 256, (Q, K // 2), generator=g, dtype=torch.uint8)
    raw = b.fp4_gemm(L.cuda(), None, R.cuda(), None).cpu()
    assert torch.equal(raw.double(), _values(L).double() @ _values(R).double().t())
    gl, gr, addend = torch.rand(P, generator=g) + 0.5, torch.rand(Q, generator=g) + 0.5, torch.randn(P, Q, generator=g)
    Pb, Qb = 3072, 3072
    Lb, Rb = torch.zeros(Pb, K // 2, dtype=torch.uint8), torch.zeros(Qb, K // 2, dtype=torch.uint8)
    Lb[:P], Rb[:Q] = L, R
    glb, grb, ab = torch.ones(Pb), torch.ones(Qb), torch.zeros(Pb, Qb)
    glb[:P], grb[:Q], ab[:P, :Q] = gl, gr, addend
    for dt in (torch.float32, torch.bfloat16):
        for a, ba in ((None, None), (addend.cuda(), ab.cuda())):
            one = b.fp4_gemm(L.cuda(), gl.cuda(), R.cuda(), gr.cuda(), out_dtype=dt, addend=a)
            big = b.fp4_gemm(Lb.cuda(), glb.cuda(), Rb.cuda(), grb.cuda(), out_dtype=dt, addend=ba)
            assert torch.equal(one, big[:P, :Q])


@pytest.mark.parametrize("K", [116480, 116512])
def test_the_longest_exact_sums(K):
    """Rows of sixes, whose sums are the largest there are: 2^22 is not reached up to 116508 codes, and the next length goes to another tiling."""
    from paper_2501_17116_amd import binding as b
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus != 256 or b.fp4_gemm_splits(33, 40, K) == (K == 116480)
    g = torch.Generator().manual_seed(K)
    L, R = (torch.randint(0, 256, (n, K // 2), generator=g, dtype=torch.uint8) for n in (33, 40))
    L[5], R[7], R[8] = 0x77, 0x77, 0xff
    exact = _values(L).double() @ _values(R).double().t()
    got = b.fp4_gemm(L.cuda(), None, R.cuda(), None).cpu().double()
    if K == 116480:
        assert exact[5, 7] == 36 * K and exact[5, 8] == -36 * K
        assert torch.equal(got, exact)
    else:   # half an ulp beyond 2^22 for each 64 codes that are added at a time
        assert torch.all((got - exact).abs() <= K / 64 * 0.25)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,K,N", [(256, 32, 32), (288, 72, 136), (512, 512, 1024), (1056, 1032, 488), (4096, 264, 520)])
def test_factor(M, K, N, dtype):
    """The weight gradient against its parts called one by one: the product is the same to the last bit, the factor one
    rounding of fp32 in either."""
    from paper_2501_17116_amd import binding as b
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus != 256 or b.fp4_gemm_splits(K, N, M, True) == (K != 1032)
    torch.manual_seed(M + N)
    A, W, dY = (t.to(dtype) for t in (torch.randn(M, K, device="cuda"), torch.randn(K, N, device="cuda") * 0.02, torch.randn(M, N, device="cuda")))
    _, ctx = b.fp4_linear_fwd(A[:, :K // 32 * 32].contiguous(), W[:K // 32 * 32].contiguous(), 1.0)
    got = b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0)
    qA, gA = b.fp4_quantize(A, b.FP4_AXIS_COL)
    qY, gY = b.fp4_quantize(dY, b.FP4_AXIS_COL)
    ref = b.fp4_dge_apply(b.fp4_gemm(qA, gA, qY, gY), W, ctx.gamma_W, 5.0, 3.0)
    assert torch.all((got - ref).abs() <= 2.0 ** -22 * ref.abs())
