"""The fp32 residual product (csrc/spmm.hip) with 512 and 1024 rows a workgroup: at the edges of the rows, of the slabs
of 512 rows of D, of the 64 columns, and on both sides of the 256 workgroups where the shape changes.

Bound: n products summed in fp32 one after another differ from the exact sum by at most n * 2^-24 * sum |v d| to first order;
2^-23 leaves room for the higher orders.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,Q,N", [(1, 1, 8), (511, 512, 72), (513, 513, 64), (512, 1030, 136), (1025, 96, 200), (2049, 520, 2048),
                                   (4096, 130, 2048), (4097, 130, 2048), (5000, 600, 1032)])   # 256 workgroups of 512 rows; more
def test_against_fp64(P, Q, N):
    from paper_2501_17116_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(P + Q + N)
    S = torch.randn(P, Q, generator=g, device="cuda") * (torch.rand(P, Q, generator=g, device="cuda") < (0.04 if P > 1 else 2.0))
    if P > 1:
        S[P // 2] = 0.0
    D = torch.randn(Q, N, generator=g, device="cuda")
    nz = S != 0
    ptr = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(nz.sum(1), 0, out=ptr[1:])
    R = torch.full((P, N), float("nan"), device="cuda")
    b.fp4_residual_spmm(ptr, nz.nonzero()[:, 1].int().contiguous(), S[nz].contiguous(), Q, D, R=R)
    ref = S.double() @ D.double()
    mag = S.double().abs() @ D.double().abs()
    n = nz.sum(1, keepdim=True).double() + 1
    assert torch.all((R.double() - ref).abs() <= n * 2.0 ** -23 * mag)


def test_no_columns():
    """A matrix without columns: zeros."""
    from paper_2501_17116_amd import binding as b
    R = torch.full((300, 64), float("nan"), device="cuda")
    ptr = torch.zeros(301, dtype=torch.int64, device="cuda")
    b.fp4_residual_spmm(ptr, torch.empty(0, dtype=torch.int32, device="cuda"), torch.empty(0, device="cuda"), 0,
                        torch.ones(1, 64, device="cuda"), R=R)
    assert torch.all(R == 0)
