"""The packed residual product (csrc/spmm_mfma.hip) in each of its workgroups' shapes: at 64 column blocks, the largest and the smallest row
count that takes 128, 192, 256, 384 and 528 rows a workgroup, with bundles that its packing or its sums leave to the tiled kernel."""
import pytest
import torch

from test_gpu_spmm_mfma import _csr, _draw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [127, 512, 513, 768, 769, 1024, 1025, 1536, 1537])
@pytest.mark.parametrize("terms", [1, 3])
def test_against_fp64(P, terms):
    from paper_2501_17116_amd import binding as b
    Q, N = 389, 8184
    S, D = _draw(P, Q, N, 0.03, terms, P + terms)
    g = torch.Generator().manual_seed(P)
    r0 = P // 2 // 16 * 16
    S[r0:r0 + 16] = torch.randn(16, Q, generator=g) * (torch.rand(16, Q, generator=g) < 0.23)   # more slots than there is room for, just not long
    S[P - 1, 7], S[:P - 1, 7] = 1.5, 0.0
    D[7, 3] = float("inf")   # reaches the last row alone, and its group's sums
    R = torch.full((P, N), float("nan"), device="cuda")
    b.fp4_residual_spmm_general(*_csr(S), Q, D.cuda(), R=R)
    got, S, D = R.double(), S.cuda().double(), D.cuda().double()
    assert got[P - 1, 3] == float("inf")
    D[7, 3], got[P - 1, 3] = 0.0, S[P - 1] @ D.nan_to_num(posinf=0.0)[:, 3]
    # n products, each exact before the sum, summed in fp32 in any order: n 2^-24 sum |v d|, twice that for the higher orders
    n = (S != 0).sum(1, keepdim=True) + 1
    assert torch.all((got - S @ D).abs() <= n * 2.0 ** -23 * (S.abs() @ D.abs()) + 1e-38)
