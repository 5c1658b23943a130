"""The gathering kernel of small residual products (csrc/spmm_gather.hip) at the edges of its rows a workgroup, its strips of columns, its
64 entries a turn and 8 or 16 a request, with rows that all waves share, and on both sides of the line where the other kernels begin.

Bound: n products summed in fp32 in any order differ from the exact sum by at most n * 2^-24 * sum |v d| to first order (those of bf16
values with up to three terms are exact, others rounded once in the FMA); 2^-23 leaves room for the higher orders.
"""
import pytest
import torch

from paper_2501_17116_amd import binding as b

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("P,Q,N", [(1, 1, 8), (7, 63, 248), (8, 64, 256), (9, 65, 264), (33, 300, 520), (1023, 129, 264), (1025, 512, 520),
                                   (2049, 96, 136), (300, 8192, 72), (40, 8193, 72),   # the widest it takes, and the next
                                   (2048, 2048, 2048), (2049, 2048, 2048)])           # 2^33, and more
def test_against_fp64(P, Q, N, dtype):
    g = torch.Generator(device="cuda").manual_seed(P + Q + N)
    S = torch.randn(P, Q, generator=g, device="cuda") * (torch.rand(P, Q, generator=g, device="cuda") < 0.05)
    if P > 5:
        S[P // 2] = 0.0                                                # an empty row
        S[P // 3] = torch.randn(Q, generator=g, device="cuda")         # rows that all waves share, two of them neighbours
        S[P // 3 + 1] = torch.randn(Q, generator=g, device="cuda")
        S[P - 1] = torch.randn(Q, generator=g, device="cuda")
    nz = S != 0
    ptr = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(nz.sum(1), 0, out=ptr[1:])
    col, val = nz.nonzero()[:, 1].int().contiguous(), S[nz].contiguous()
    D = torch.randn(Q, N, generator=g, device="cuda").to(dtype)
    R = torch.full((P, N), float("nan"), device="cuda")
    b.fp4_residual_spmm(ptr, col, val, Q, D, R=R)
    mag = S.double().abs() @ D.double().abs()
    n = nz.sum(1, keepdim=True).double() + 1
    assert torch.all((R.double() - S.double() @ D.double()).abs() <= n * 2.0 ** -23 * mag)
    assert torch.equal(R, b.fp4_residual_spmm(ptr, col, val, Q, D))    # a fixed order
    assert torch.all((R - b.fp4_residual_spmm_general(ptr, col, val, Q, D)).abs() <= 2 * n * 2.0 ** -23 * mag)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_entries_in_any_order(dtype):
    """Columns unsorted and repeated, a first entry that is not the array's first."""
    g = torch.Generator(device="cuda").manual_seed(3)
    P, Q, N = 50, 200, 264
    count = torch.randint(0, 90, (P,), generator=g, device="cuda")
    ptr = torch.full((P + 1,), 11, dtype=torch.int64, device="cuda")
    ptr[1:] += torch.cumsum(count, 0)
    nnz = int(ptr[-1])
    col = torch.randint(0, Q, (nnz,), generator=g, device="cuda").int()
    val = torch.randn(nnz, generator=g, device="cuda")
    D = torch.randn(Q, N, generator=g, device="cuda").to(dtype)
    row = torch.repeat_interleave(torch.arange(P, device="cuda"), count)
    ref = torch.zeros(P, N, dtype=torch.float64, device="cuda").index_add_(0, row, val[11:, None].double() * D.double()[col[11:].long()])
    mag = torch.zeros_like(ref).index_add_(0, row, (val[11:, None].double() * D.double()[col[11:].long()]).abs())
    R = b.fp4_residual_spmm(ptr, col, val, Q, D)
    assert torch.all((R.double() - ref).abs() <= (count[:, None] + 1).double() * 2.0 ** -23 * mag)


def _csr(mask, g):
    ptr = torch.zeros(mask.shape[0] + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(mask.sum(1), 0, out=ptr[1:])
    S = torch.randn(*mask.shape, generator=g, device="cuda").bfloat16().float()
    return ptr, mask.nonzero()[:, 1].int().contiguous(), S[mask].contiguous()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("apart", [1, 8, 16, 64, 128])
def test_full_rows_at_a_distance_cost_what_one_does(apart, dtype):
    """Eight of them, side by side or a head's width apart, are eight workgroups' (side by side and taken one after another by one, they
    cost 2.3 times as much as a single one)."""
    P, Q, N = 2048, 2048, 1024
    g = torch.Generator(device="cuda").manual_seed(1)
    sparse = torch.rand(P, Q, generator=g, device="cuda") < 0.01
    D = torch.randn(Q, N, generator=g, device="cuda").to(dtype)
    R = torch.empty(P, N, device="cuda")
    best = []
    for rows in (1, 8):
        mask = sparse.clone()
        mask[[1024 - 4 * apart + i * apart for i in range(rows)]] = True
        args = _csr(mask, g)
        for _ in range(3):
            b.fp4_residual_spmm(*args, Q, D, R=R)
        times = []
        for _ in range(12):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(8):
                b.fp4_residual_spmm(*args, Q, D, R=R)
            e[1].record()
            e[1].synchronize()
            times.append(e[0].elapsed_time(e[1]))
        best.append(min(times))
    assert best[1] < 2.0 * best[0], best


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("P,Q,N", [(40, 600, 136), (1030, 300, 520)])   # a row a workgroup, eight rows
def test_infinities_and_nan_stay_with_their_entries(P, Q, N, dtype):
    """Rows of D that are not finite reach the rows of S with an entry there, and no others: not those of the same workgroup or wave, not
    rows that all waves share, and not through the zeros that fill a request up."""
    g = torch.Generator(device="cuda").manual_seed(P)
    mask = torch.rand(P, Q, generator=g, device="cuda") < 0.02
    mask[P // 3] = True
    mask[P // 3, 5:8] = False            # a long row without an entry in the rows that are not finite
    mask[P // 2] = True
    ptr, col, val = _csr(mask, g)
    D = torch.randn(Q, N, generator=g, device="cuda")
    D[5, ::3] = float("inf")
    D[6, 1::3] = -float("inf")
    D[7, 2::5] = float("nan")
    D = D.to(dtype)
    assert b.fp4_residual_spmm_gathers(P, Q, N, b.FP4_BF16 if dtype == torch.bfloat16 else b.FP4_F32, col.numel())
    R = b.fp4_residual_spmm(ptr, col, val, Q, D)
    row = torch.repeat_interleave(torch.arange(P, device="cuda"), ptr[1:] - ptr[:-1])
    ref = torch.zeros(P, N, dtype=torch.float64, device="cuda").index_add_(0, row, val[:, None].double() * D.double()[col.long()])
    mag = torch.zeros_like(ref).index_add_(0, row, (val[:, None].double() * D.double()[col.long()]).abs())
    assert torch.equal(R.isnan(), ref.isnan())
    infinite = ref.isinf()
    assert torch.equal(R[infinite].double(), ref[infinite])
    fine = ref.isfinite()
    n = (ptr[1:] - ptr[:-1])[:, None].double() + 1
    assert torch.all(((R.double() - ref).abs() <= n * 2.0 ** -23 * mag)[fine])
    assert fine[P // 3].all() and not fine[P // 2].all()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("P,Q,N,full", [(5, 4104, 8, [4]), (3, 4104, 72, [1]), (70, 4104, 136, [0, 1, 69]), (600, 4160, 520, [7, 8, 9, 400, 599]),
                                        (1200, 6000, 72, list(range(0, 1200, 97))),
                                        (64, 4608, 8192, [1, 3, 8, 9, 10, 30, 62, 63])])   # more full rows than there are workgroups for a strip
def test_long_rows_of_more_than_4096_columns(P, Q, N, full, dtype):
    """Rows that the first workgroups take, beside rows that a workgroup's waves share (between four times the mean and 256 entries) and others."""
    g = torch.Generator(device="cuda").manual_seed(P + Q)
    mask = torch.rand(P, Q, generator=g, device="cuda") < 4.0 / Q
    mask[P // 2] = torch.rand(Q, generator=g, device="cuda") < 120.0 / Q
    for r in full:
        mask[r] = torch.rand(Q, generator=g, device="cuda") < (0.9 if r % 2 else 300.0 / Q)
    ptr, col, val = _csr(mask, g)
    D = torch.randn(Q, N, generator=g, device="cuda").to(dtype)
    assert b.fp4_residual_spmm_gathers(P, Q, N, b.FP4_BF16 if dtype == torch.bfloat16 else b.FP4_F32, col.numel())
    R = torch.full((P, N), float("nan"), device="cuda")
    b.fp4_residual_spmm(ptr, col, val, Q, D, R=R)
    row = torch.repeat_interleave(torch.arange(P, device="cuda"), ptr[1:] - ptr[:-1])
    S = torch.zeros(P, Q, dtype=torch.float64, device="cuda")
    S[row, col.long()] = val.double()
    n = (ptr[1:] - ptr[:-1])[:, None].double() + 1
    assert torch.all((R.double() - S @ D.double()).abs() <= n * 2.0 ** -23 * (S.abs() @ D.double().abs()))
    assert torch.equal(R, b.fp4_residual_spmm(ptr, col, val, Q, D))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_a_full_row_of_8192_columns_is_not_waited_for(dtype):
    """One among 1 %: a few workgroups that took it as it came, a wide strip each, made the product five to eight times as long."""
    P, Q, N = 512, 8192, 512
    g = torch.Generator(device="cuda").manual_seed(1)
    mask = torch.rand(P, Q, generator=g, device="cuda") < 0.01
    D = torch.randn(Q, N, generator=g, device="cuda").to(dtype)
    R = torch.empty(P, N, device="cuda")
    best = []
    for full in (False, True):
        mask[P // 3] |= full
        args, ws = _csr(mask, g), b.Workspace()
        graph = torch.cuda.CUDAGraph()
        b.fp4_residual_spmm(*args, Q, D, R=R, ws=ws)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            for _ in range(8):
                b.fp4_residual_spmm(*args, Q, D, R=R, ws=ws)
        times = []
        for _ in range(12):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            graph.replay()
            e[1].record()
            e[1].synchronize()
            times.append(e[0].elapsed_time(e[1]))
        best.append(min(times))
    assert best[1] < 4.2 * best[0], best
