"""The FP4 GEMM's small-tile kernel at the edges of its tiles and of the rule that selects it: against the exact
integer product (raw accumulators) and, scaled, bit for bit against a problem large enough for the 256 x 256 tiles that
holds the same rows and columns."""
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
