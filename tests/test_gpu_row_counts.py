"""Thresholds and residual of the clamp where the row counts take another route: windows behind an exact digit (bf16, up to 2^25
elements), rows counted from their elements (a NaN; zeros that are outliers), block sums in the emitting kernel (up to 65536 rows; two,
four or eight rows a wave from 8192, 16384 and 32768) or a scan beyond."""
import numpy as np
import pytest
import torch

from paper_2501_17116_amd import binding as b
from test_gpu_select import _compare, _one_sided

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", ["normal", "relu", "masked", "relu_neg", "sparse", "one value", "two values", "row scales"])
@pytest.mark.parametrize("rows,cols,alpha", [(1, 504, 0.99), (16, 504, 0.99), (64, 2048, 0.99), (1056, 1376, 0.97), (2049, 1032, 0.999)])
def test_windows_behind_an_exact_digit(rows, cols, alpha, what):
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = _one_sided(what, rows, cols, alpha, g)
    for _ in range(2):
        _compare(b.occ_clamp_residual(x, alpha), x, alpha)


@pytest.mark.parametrize("what", ["some", "most negative", "all of one pattern", "just above zero", "just below zero"])
def test_rows_that_their_bins_do_not_count(what):
    rows, cols, alpha = 264, 1032, 0.99
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(rows, cols, generator=g, device="cuda").bfloat16()
    bits = x.view(torch.int16)
    if what == "some":
        bits[5, 17::7] = 0x7FC0
        bits[9, 3::50] = -64            # 0xffc0
    elif what == "most negative":       # more than k of the lowest key: the threshold is that pattern
        bits[:, ::40] = -1
    elif what == "all of one pattern":
        bits[:] = -1
    else:
        u = torch.rand(rows, cols, generator=g, device="cuda")
        y = torch.where(u < 0.03, torch.full_like(u, 2.0 ** -130), x.float().abs() + 0.5)
        y = torch.where(u < 0.004, torch.zeros_like(y), y)
        x = (y if what == "just above zero" else -y).bfloat16()
        bits = x.view(torch.int16)
    k = int(np.floor((1.0 - alpha) * x.numel()))
    key = bits.flatten().int()
    key = torch.where(key < 0, -32769 - key, key).sort().values
    want = torch.stack([key[k], key[x.numel() - 1 - k]])
    want = torch.where(want < 0, -32769 - want, want).short()
    out = b.occ_clamp_residual(x, alpha)
    assert torch.equal((out["thresholds"].view(torch.int32) >> 16).short(), want)
    lo, hi = want.view(torch.bfloat16).float()
    counts = ((x.float() < lo) | (x.float() > hi)).sum(1)       # NaN compares false
    assert torch.equal(out["row_ptr"][1:] - out["row_ptr"][:-1], counts)
    assert int(out["nnz"]) == int(counts.sum())


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,cols", [(5, 96), (8192, 64), (8193, 64), (16388, 32), (32769, 32), (65536, 32), (65537, 32), (40, 16392)])
def test_row_pointers(rows, cols, dtype):
    alpha = 0.97
    g = torch.Generator(device="cuda").manual_seed(cols)
    x = (torch.randn(rows, cols, generator=g, device="cuda") * torch.rand(rows, 1, generator=g, device="cuda")).to(dtype)
    flat = x.float().flatten().sort().values
    k = int(np.floor((1.0 - alpha) * x.numel()))
    lo, hi = flat[k], flat[x.numel() - 1 - k]
    outlier = (x.float() < lo) | (x.float() > hi)
    out = b.occ_clamp_residual(x, alpha)
    want = torch.zeros(rows + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(outlier.sum(1), 0, out=want[1:])
    assert torch.equal(out["row_ptr"], want)
    n = int(want[-1])
    assert int(out["nnz"]) == n
    assert torch.equal(out["col_idx"][:n].long(), outlier.nonzero()[:, 1])
    rest = x.float() - x.float().clamp(lo, hi)
    assert torch.equal(out["val"][:n], rest[outlier])
