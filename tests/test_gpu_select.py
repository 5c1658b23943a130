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


@pytest.mark.parametrize("what", ["normal", "channels", "constant", "zeros", "nan", "misled"])
@pytest.mark.parametrize("rows,cols,alpha", [(8192, 4096, 0.99), (8192, 4096, 0.999), (4104, 8184, 0.97), (4104, 8184, 0.9)])
def test_large_tensors(rows, cols, alpha, what):
    """Thresholds and row counts out of one pass, and what makes it give up: windows that meet, thresholds of zero, a NaN, a
    sample (128 runs of 16384 elements, evenly spaced) that is not like the rest."""
    from paper_2501_17116_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = torch.randn(rows, cols, generator=g, device="cuda")
    if what == "channels":
        x[:, ::997] *= 50
    elif what == "constant":
        x = torch.full_like(x, -1.5)
    elif what == "zeros":
        x = torch.where(torch.rand(rows, cols, generator=g, device="cuda") < 0.02 * (1 - alpha), x, torch.copysign(torch.zeros_like(x), x))
    elif what == "nan":
        x[5, 17::7] = float("nan")
    elif what == "misled":
        n = rows * cols // 8
        at = (torch.arange(128, device="cuda")[:, None] * (n - 2048) // 127 + torch.arange(2048, device="cuda")).reshape(-1)
        x.view(-1, 8)[at] *= 2.0 ** 20
    x = x.bfloat16()
    k = int(np.floor((1.0 - alpha) * (rows * cols)))
    flat = x.float().flatten().sort().values
    lo, hi = flat[k].item(), flat[rows * cols - 1 - k].item()
    out = b.occ_clamp_residual(x, alpha)
    assert out["thresholds"].cpu().tolist() == [lo, hi]
    counts = ((x.float() < lo) | (x.float() > hi)).sum(1)
    assert torch.equal(out["row_ptr"][1:] - out["row_ptr"][:-1], counts)
