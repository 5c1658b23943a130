"""Threshold selection (csrc/occ.hip) at the sizes where its launches change: one workgroup, two, the last count of them that
picks the bins inside the digit pass, the first that does not, and the most before a workgroup's share grows."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,cols", [(1, 32), (8, 1024), (8, 1032), (64, 2048), (512, 1024), (513, 1024), (2048, 1024), (2049, 1032)])
def test_thresholds_are_the_order_statistics(rows, cols, dtype):
    from paper_2501_17116_amd import binding as b
    g = torch.Generator().manual_seed(rows * cols)
    x = (torch.randn(rows, cols, generator=g) * torch.exp2(torch.randint(-8, 9, (rows, 1), generator=g).float())).to(dtype)
    k = int(np.floor((1.0 - 0.99) * (rows * cols)))
    flat = x.float().flatten().sort().values
    xd = x.cuda()
    for _ in range(2):   # the state left by a call must not reach the next
        thr = b.occ_clamp_residual(xd, 0.99)["thresholds"]
        assert thr.cpu().tolist() == [flat[k].item(), flat[rows * cols - 1 - k].item()]
