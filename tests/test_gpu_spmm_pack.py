"""The packing of the matrix-core residual product on either side of the number of bundles up to which a workgroup writes one group of a
bundle (170 of 48 rows on 256 CUs), with a last bundle that is not whole.  Bound as in test_gpu_spmm_gather.py."""
import pytest
import torch

from paper_2501_17116_amd import binding as b

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("terms", [1, 3])
@pytest.mark.parametrize("P", [8159, 8161, 8193])
def test_against_fp64(P, terms):
    Q, N = 264, 2056
    g = torch.Generator(device="cuda").manual_seed(P)
    S = torch.randn(P, Q, generator=g, device="cuda") * (torch.rand(P, Q, generator=g, device="cuda") < 0.02)
    if terms == 1:
        S = S.bfloat16().float()
    nz = S != 0
    ptr = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(nz.sum(1), 0, out=ptr[1:])
    col, val = nz.nonzero()[:, 1].int().contiguous(), S[nz].contiguous()
    D = torch.randn(Q, N, generator=g, device="cuda").bfloat16()
    R = b.fp4_residual_spmm_general(ptr, col, val, Q, D)
    n = nz.sum(1, keepdim=True).double() + 1
    assert torch.all((R.double() - S.double() @ D.double()).abs() <= n * 2.0 ** -23 * (S.double().abs() @ D.double().abs()))
