"""The bf16 residual product on the matrix cores (csrc/spmm_mfma.hip) where its packing and tiling can go wrong:
row and column counts around its tiles, chunk edges, values of one to three bf16 terms, rows it leaves to the
long-row kernels, bundles it leaves to the tiled kernel, non-finite elements.

Bound: n products summed in fp32 in any order, each exact before the sum, differ from the exact sum by at most
n * 2^-24 * sum |v d| to first order; 2^-23 leaves room for the higher orders and the matrix core's own adder.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _csr(S):
    nz = S != 0
    row_ptr = torch.zeros(S.shape[0] + 1, dtype=torch.int64)
    torch.cumsum(nz.sum(1), 0, out=row_ptr[1:])
    idx = nz.nonzero()
    return row_ptr.cuda(), idx[:, 1].int().contiguous().cuda(), S[nz].contiguous().cuda()


def _check(S, D, rows=None):
    from paper_2501_17116_amd import binding as b
    R = torch.full((S.shape[0], D.shape[1]), float("nan"), device="cuda")
    b.fp4_residual_spmm(*_csr(S), S.shape[1], D.cuda(), R=R)
    got = R.cpu().double()
    ref = S.double() @ D.double()
    mag = S.double().abs() @ D.double().abs()
    n = (S != 0).sum(1, keepdim=True).double() + 1
    sel = slice(None) if rows is None else rows
    assert torch.all((got - ref).abs()[sel] <= (n * 2.0 ** -23 * mag + 1e-38)[sel])
    return R


def _draw(P, Q, N, density, terms, seed):
    g = torch.Generator().manual_seed(seed)
    S = torch.randn(P, Q, generator=g) * (torch.rand(P, Q, generator=g) < density)
    if terms == 1:
        S = S.bfloat16().float()
    elif terms == 2:
        S = S.bfloat16().float() - (S != 0) * 0.7109375 * 2.0 ** -7
    return S, (torch.randn(Q, N, generator=g) * 0.02).bfloat16()


@pytest.mark.parametrize("P,Q,N,density,terms", [
    (1, 32, 8, 0.5, 1), (16, 128, 128, 0.02, 1), (17, 129, 136, 0.05, 3), (112, 127, 120, 0.1, 2),
    (113, 256, 264, 0.02, 3), (176, 640, 128, 0.3, 1), (177, 641, 248, 0.3, 2), (528, 1376, 2080, 0.06, 2),
    (529, 768, 4104, 0.02, 1), (1057, 96, 16392, 0.02, 1), (4096, 2100, 1032, 0.002, 2), (64, 4096, 512, 0.02, 1),
    (40, 24576, 72, 0.002, 2), (40, 24608, 72, 0.002, 2),   # the widest that is packed, and the next
])
def test_against_fp64(P, Q, N, density, terms):
    _check(*_draw(P, Q, N, density, terms, P + Q + N))


@pytest.mark.parametrize("density,terms", [(0.0, 1), (1.0, 1), (1.0, 3)])
def test_empty_and_full(density, terms):
    _check(*_draw(200, 700, 136, density, terms, 5))


@pytest.mark.parametrize("P,N", [(700, 520), (4500, 4104)])
def test_bundles_without_room_beside_packed_ones(P, N):
    """Groups whose three-term values take more slots than there is room for, in a matrix that is worth packing: the tiled
    kernel writes their rows (one workgroup's, and in several), the packed product the others'."""
    S, D = _draw(P, 1300, N, 0.01, 1, 29)
    g = torch.Generator().manual_seed(29)
    for r0 in (32, P - 20):
        rows = slice(r0, min(r0 + 16, P))
        n = S[rows].shape[0]
        S[rows] = torch.randn(n, 1300, generator=g) * (torch.rand(n, 1300, generator=g) < 0.23)   # just not long
    R = _check(S, D)
    few = S.clone()
    few[32:48] = 0
    few[P - 20:P - 4] = 0
    from paper_2501_17116_amd import binding as b
    far = slice(96, P - 100)   # other bundles: the same bits whatever their neighbours hold
    assert torch.equal(b.fp4_residual_spmm(*_csr(few), 1300, D.cuda())[far], R[far])


@pytest.mark.parametrize("scope", [0, 1])
def test_spare_capacity_changes_nothing(scope):
    """Residual buffers larger than the clamp needs (as for alpha = 0.9): the same kernels, the same bits."""
    from paper_2501_17116_amd import binding as b
    torch.manual_seed(7)
    M, K, N = 512, 768, 520 + 24
    A = torch.randn(M, K, device="cuda")
    A[:, 5] *= 30
    A, W, dY = A.bfloat16(), (torch.randn(K, N, device="cuda") * 0.02).bfloat16(), (torch.randn(M, N, device="cuda") * 0.01).bfloat16()
    out = []
    for alpha in (0.99, 0.9):
        ctx = b.FwdCtx(M, K, N, alpha, scope=scope)
        Y, _ = b.fp4_linear_fwd(A, W, 0.99, ctx=ctx)
        out.append((Y, *b.fp4_linear_bwd(dY, A, W, ctx, 5.0, 3.0), b.fp4_linear_bwd_wgrad(A, dY, W, ctx, 5.0, 3.0)))
    for x, y in zip(*out):
        assert torch.equal(x, y)


def test_long_rows_and_dense_columns():
    S, D = _draw(300, 4096, 264, 0.01, 2, 9)
    S[7] = torch.randn(4096)              # left to the long-row kernels
    S[40, :2048] = torch.randn(2048).bfloat16().float()   # just not
    S[:, 1000] = torch.randn(300)
    S[:, 1001] = torch.randn(300) * 50
    _check(S, D)


def test_extreme_magnitudes():
    S, D = _draw(50, 300, 72, 0.1, 1, 11)
    S *= torch.exp2(torch.randint(-100, 60, S.shape, generator=torch.Generator().manual_seed(1)).float())
    _check(S, D)


@pytest.mark.parametrize("terms", [2, 3])
@pytest.mark.parametrize("exp", [-149, -126, -118, -111, -104, 0, 120, 126])
def test_split_of_extreme_values(terms, exp):
    """Values around 2^exp, of every bit fp32 has there, against columns of D that bring the products to the middle of
    the range: the sum of the bf16 terms has to be the value itself (below 2^-110 three of them are not enough)."""
    from paper_2501_17116_amd import binding as b
    S, D = _draw(64, 300, 72, 0.02, terms, 11 + terms)   # few enough slots for the packed path
    S = (S.double() * 2.0 ** exp).clamp(-3.4e38, 3.4e38).float()
    D = (D.double() * 2.0 ** max(-100, min(100, -exp))).bfloat16()
    if exp > 100:
        S[7, :40] = torch.tensor([3.4028234e38, -3.4028234e38, 3.3961776e38, 3.39e38]).repeat(10)
    got = b.fp4_residual_spmm(*_csr(S), 300, D.cuda()).cpu().double()
    ref, mag = S.double() @ D.double(), S.double().abs() @ D.double().abs()
    n = (S != 0).sum(1, keepdim=True).double() + 1
    # 2^-23 as above; results of subnormal size carry half a unit of 2^-149 per sum besides
    assert torch.all((got - ref).abs() <= n * 2.0 ** -23 * mag + n * 2.0 ** -150)


@pytest.mark.parametrize("exp_s,exp_d", [(-60, -70), (-100, -30), (0, -126), (0, -132), (-100, 0)])
def test_tiny_products(exp_s, exp_d):
    """Products and elements of D near and below the smallest normal numbers."""
    from paper_2501_17116_amd import binding as b
    S, D = _draw(64, 300, 72, 0.02, 2, 23)
    S = (S.double() * 2.0 ** exp_s).float()
    D = (D.double() * 2.0 ** exp_d).bfloat16()
    got = b.fp4_residual_spmm(*_csr(S), 300, D.cuda()).cpu().double()
    ref, mag = S.double() @ D.double(), S.double().abs() @ D.double().abs()
    n = (S != 0).sum(1, keepdim=True).double() + 1
    # up to three products an entry, each sum rounded to 2^-149 at the finest
    assert torch.all((got - ref).abs() <= n * 2.0 ** -23 * mag + 3 * n * 2.0 ** -150)


def test_non_finite_elements_stay_in_their_rows():
    from paper_2501_17116_amd import binding as b
    S, D = _draw(64, 400, 136, 0.05, 1, 13)
    S[:, 100] = 0
    S[:, 200] = 0
    S[5, 100], S[33, 200] = 1.5, -2.0
    D[100, 10], D[200, 100] = float("inf"), float("nan")
    D[300] = 0
    S[20, 300] = float("inf")             # inf * 0
    R = torch.empty(64, 136, device="cuda")
    b.fp4_residual_spmm(*_csr(S), 400, D.cuda(), R=R)
    got = R.cpu()
    assert got[5, 10] == float("inf") and torch.isnan(got[33, 100]) and torch.isnan(got[20]).all()
    bad = torch.zeros(64, 136, dtype=torch.bool)
    bad[5, 10] = bad[33, 100] = True
    bad[20] = True
    assert torch.isfinite(got[~bad]).all()
    clean = S.clone(); clean[20] = 0
    Dc = D.clone(); Dc[100, 10] = 0; Dc[200, 100] = 0
    ref, mag = clean.double() @ Dc.double(), clean.double().abs() @ Dc.double().abs()
    n = (S != 0).sum(1, keepdim=True).double() + 1
    assert torch.all((((got.double() - ref).abs() <= n * 2.0 ** -23 * mag + 1e-38) | bad))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("long_rows", [[3, 50, 51, 120], list(range(0, 190, 5))])
def test_non_finite_elements_stay_out_of_long_rows_without_them(dtype, long_rows):
    """A long row that has no entry in an infinite element's row of D is finite; one that has, is infinite there only.  Four
    long rows, and more than the 32 up to which a span of D is one slice."""
    from paper_2501_17116_amd import binding as b
    S, D = _draw(200, 600, 520, 0.01, 1, 19)
    g = torch.Generator().manual_seed(19)
    for r in long_rows:
        S[r] = torch.randn(600, generator=g)
    S[:, 333] = 0
    S[:, 90] = 0
    S[50, 333], S[120, 90] = 2.0, -1.0
    S[185, 333] = 3.0
    D = D.to(dtype)
    D[333, 40], D[90, 400] = float("inf"), float("nan")
    got = b.fp4_residual_spmm(*_csr(S), 600, D.cuda()).cpu()
    bad = torch.zeros(200, 520, dtype=torch.bool)
    bad[50, 40] = bad[120, 400] = bad[185, 40] = True
    assert got[50, 40] == got[185, 40] == float("inf") and torch.isnan(got[120, 400])
    Df = D.double()
    Df[333, 40] = Df[90, 400] = 0
    ref, mag = S.double() @ Df, S.double().abs() @ Df.abs()
    n = (S != 0).sum(1, keepdim=True).double() + 1
    assert torch.all(((got.double() - ref).abs() <= n * 2.0 ** -23 * mag + 1e-38) | bad)


def test_repeated_columns_are_summed():
    from paper_2501_17116_amd import binding as b
    D = torch.randn(64, 16).bfloat16()
    rp = torch.tensor([0, 3, 5]).cuda()
    ci = torch.tensor([4, 4, 9, 0, 63], dtype=torch.int32).cuda()
    v = torch.tensor([1.0, 2.0, -1.0, 0.5, 4.0]).cuda()
    R = b.fp4_residual_spmm(rp, ci, v, 64, D.cuda()).cpu()
    Df = D.float()
    assert np.allclose(R[0], 3 * Df[4] - Df[9], rtol=1e-6, atol=1e-6) and np.allclose(R[1], 0.5 * Df[0] + 4 * Df[63], rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("Q", [32, 64, 65, 256, 700])
def test_repeated_columns_in_rows_above_the_long_limit(Q, dtype):
    """Rows of more entries than a row of distinct columns could have (Q <= 64: no row is long), and rows that count as
    long (more than max(64, Q / 4) entries) with repeats inside a slice, on its edges and of a whole slice's columns."""
    from paper_2501_17116_amd import binding as b
    g = torch.Generator().manual_seed(Q)
    rows = [torch.arange(0)] * 400
    for r in range(50, 400, 9):   # more long rows (where there are any) than the 32 up to which a span is one slice
        rows[r] = torch.randint(0, Q, (350,), generator=g).sort().values
    rows[3] = torch.arange(Q).repeat_interleave(3)                                   # every column three times
    rows[17] = torch.cat([torch.arange(min(Q, 90)), torch.tensor([min(Q, 90) - 1])])   # one repeat, on the last column
    rows[18] = torch.cat([torch.zeros(70, dtype=torch.long), torch.arange(Q)])
    rows[30] = torch.randint(0, Q, (300,), generator=g).sort().values
    rows[39] = torch.randint(0, Q, (5,), generator=g).sort().values
    rp = torch.zeros(401, dtype=torch.int64)
    torch.cumsum(torch.tensor([len(r) for r in rows]), 0, out=rp[1:])
    ci = torch.cat(rows)
    v = torch.randn(len(ci), generator=g)
    D = torch.randn(Q, 264, generator=g).to(dtype)
    S = torch.zeros(400, Q, dtype=torch.float64)
    A = torch.zeros(400, Q, dtype=torch.float64)
    at = (torch.repeat_interleave(torch.arange(400), rp.diff()), ci)
    S.index_put_(at, v.double(), accumulate=True)
    A.index_put_(at, v.double().abs(), accumulate=True)
    args = (rp.cuda(), ci.int().cuda(), v.cuda(), Q, D.cuda())
    R = torch.full((400, 264), float("nan"), device="cuda")
    b.fp4_residual_spmm(*args, R=R)
    # n products and up to as many sums of values, each rounded once: n * 2^-23 of the magnitudes, as above
    bound = (rp.diff()[:, None] + 1) * 2.0 ** -23 * (A @ D.double().abs()) + 1e-38
    assert torch.all((R.cpu().double() - S @ D.double()).abs() <= bound)
    assert torch.equal(b.fp4_residual_spmm(*args), R)


def test_same_bits_every_time():
    from paper_2501_17116_amd import binding as b
    S, D = _draw(700, 1300, 520, 0.03, 2, 17)
    c = _csr(S)
    Dd = D.cuda()
    first = b.fp4_residual_spmm(*c, 1300, Dd).clone()
    for _ in range(3):
        assert torch.equal(b.fp4_residual_spmm(*c, 1300, Dd), first)
