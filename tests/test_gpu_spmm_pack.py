"""The packing of the matrix-core residual product on either side of the number of bundles up to which a workgroup writes one group of a
bundle (170 of 48 rows on 256 CUs), with a last bundle that is not whole, for values of one term and of three.  Bound as in
test_gpu_spmm_gather.py."""
import pytest
import torch

from paper_2501_17116_amd import binding as b

pytestmark = pytest.mark.gpu


def _worth_packing(ptr, val, P, Q, N):
    """csrc/spmm_mfma.hip's pk_worth: slots a column of a group of 16 rows needs, from 64 rows and the terms of one value of each."""
    ptr, val = ptr.cpu(), val.cpu()
    rows = [int(i * P // 64) for i in range(64)]
    entries = [0.0] * 4
    for r in rows:
        b0, n = int(ptr[r]), int(ptr[r + 1] - ptr[r])
        if n == 0:
            continue
        v = val[b0 + n // 2]
        left = v - v.bfloat16().float()
        third = left - left.bfloat16().float()
        entries[1] += n
        entries[2] += n if left != 0 else 0
        entries[3] += n if third != 0 else 0
    cells = 64.0 * Q
    slots = sum(1.0 - max(1.0 - entries[t] / cells, 0.0) ** 16 for t in (1, 2, 3))
    small_grid = (P + 1023) // 1024 * ((N + 63) // 64) < 256
    return slots <= 1.15 and (small_grid or slots <= 0.14 + 21.0 * entries[1] / cells), entries


@pytest.mark.parametrize("terms", [1, 3])
@pytest.mark.parametrize("P", [8159, 8161, 8193])
def test_against_fp64(P, terms):
    Q, N = 264, 2056
    g = torch.Generator(device="cuda").manual_seed(P)
    # values of three terms take three slots a column: a matrix of 2 % would be left to the tiled kernel
    share = 0.02 if terms == 1 else 0.004
    S = torch.randn(P, Q, generator=g, device="cuda") * (torch.rand(P, Q, generator=g, device="cuda") < share)
    if terms == 1:
        S = S.bfloat16().float()
    nz = S != 0
    ptr = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(nz.sum(1), 0, out=ptr[1:])
    col, val = nz.nonzero()[:, 1].int().contiguous(), S[nz].contiguous()
    worth, entries = _worth_packing(ptr, val, P, Q, N)
    assert worth and (entries[3] > 0.8 * entries[1]) == (terms == 3), entries
    D = torch.randn(Q, N, generator=g, device="cuda").bfloat16()
    R = b.fp4_residual_spmm_general(ptr, col, val, Q, D)
    n = nz.sum(1, keepdim=True).double() + 1
    assert torch.all((R.double() - S.double() @ D.double()).abs() <= n * 2.0 ** -23 * (S.double().abs() @ D.double().abs()))
