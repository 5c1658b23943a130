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
    """Thresholds and row counts out of one pass: windows that meet, thresholds of zero, a NaN, which leaves them to the digit
    passes, and 128 runs of 16384 elements, evenly spaced, that are not like the rest."""
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


def _clamp(x, alpha):
    """occ_clamp_residual with a workspace of its own: outputs, and whether one pass gave them (SelState::done, the tenth word
    of the selection state, which lies at the workspace's start)."""
    from paper_2501_17116_amd import binding as b
    ws = b.Workspace()
    out = b.occ_clamp_residual(x, alpha, ws=ws)
    buf = ws.get(1)
    at = (-buf.data_ptr()) % 256
    return out, int(buf[at:at + 64].view(torch.int32)[9])


def _one_sided(what, rows, cols, alpha, g):
    x = torch.randn(rows, cols, generator=g, device="cuda")
    u = torch.rand(rows, cols, generator=g, device="cuda")
    if what == "relu":
        x = x.clamp_min(0)                                       # +0
    elif what == "masked":
        x = x.clamp_min(0) * (u - 0.3).sign()                    # zeros of either sign, and few negatives
        x = torch.where((x < 0) & (u < 0.29), -x, x)
    elif what == "relu_neg":
        x = -x.clamp_min(0)                                      # -0
    elif what == "squared":
        x = (x - 1.28).clamp_min(0) ** 2
    elif what == "sparse":
        x = torch.where(u < 1 - alpha, x, torch.copysign(torch.zeros_like(x), x))   # both thresholds are zeros
    elif what == "padded":
        x[: rows * 3 // 4] = 0
    elif what == "one value":
        x = torch.full_like(x, -1.5)
    elif what == "two values":
        x = torch.where(u < 0.5, 1.0, 1.25)
    elif what == "large rows":
        x[:: 100] *= 100
    elif what == "row scales":
        x *= torch.exp2(3 * torch.randn(rows, 1, generator=g, device="cuda"))
    return x.bfloat16()


def _compare(out, x, alpha):
    n = x.numel()
    k = int(np.floor((1.0 - alpha) * n))
    key = x.view(torch.int16).flatten().int()
    key = torch.where(key < 0, -32769 - key, key).sort().values   # the order of the bit patterns: -0 before +0
    want = torch.tensor([key[k], key[n - 1 - k]])
    want = torch.where(want < 0, -32769 - want, want).short().view(torch.bfloat16).float()
    thr = out["thresholds"].cpu()
    assert torch.equal(thr.view(torch.int32), want.view(torch.int32))
    xc = x.cpu().float()
    outlier = (xc < want[0]) | (xc > want[1])
    assert torch.equal((out["row_ptr"][1:] - out["row_ptr"][:-1]).cpu(), outlier.sum(1))
    m = int(out["nnz"])
    assert torch.equal(out["col_idx"][:m].cpu().long(), outlier.nonzero()[:, 1])


@pytest.mark.parametrize("what", ["relu", "masked", "relu_neg", "squared", "sparse", "padded", "one value", "two values", "large rows", "row scales"])
@pytest.mark.parametrize("rows,cols,alpha", [(8192, 4096, 0.99), (4104, 8184, 0.97), (66584, 504, 0.99)])
def test_one_pass_answers_for_what_activations_are_like(rows, cols, alpha, what):
    """Zeros as thresholds, of either sign; thresholds next to each other; a sample that few rows decide."""
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = _one_sided(what, rows, cols, alpha, g)
    for _ in range(2):
        out, done = _clamp(x, alpha)
        assert done == 1
        _compare(out, x, alpha)


@pytest.mark.parametrize("what", ["misled", "just above zero", "just below zero"])
def test_what_one_pass_leaves_to_the_digits(what):
    """A sample (4096 runs of 512 elements, evenly spaced) that is not like the rest; zeros that are outliers beside a threshold that is
    nearly one."""
    rows, cols, alpha = 8192, 4096, 0.99
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(rows, cols, generator=g, device="cuda").abs() + 0.5
    u = torch.rand(rows, cols, generator=g, device="cuda")
    if what == "misled":
        n = rows * cols // 8
        at = (torch.arange(4096, device="cuda")[:, None] * (n - 64) // 4095 + torch.arange(64, device="cuda")).reshape(-1)
        x.view(-1, 8)[at] *= 2.0 ** 20
    else:
        x = torch.where(u < 0.03, torch.full_like(x, 2.0 ** -130), x)
        x = torch.where(u < 0.004, torch.zeros_like(x), x)
        if what == "just below zero":
            x = -x
    x = x.bfloat16()
    out, done = _clamp(x, alpha)
    assert done == 0
    _compare(out, x, alpha)
