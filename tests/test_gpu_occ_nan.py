"""A NaN in a clamped tensor is no entry of the residual, whichever pass looks at it: counted and emitted entries are the same,
in their rows' segments, and nothing is written behind them."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _check(out, x, lo, hi, guard):
    x, lo, hi = x.float().cpu(), lo.cpu().reshape(-1, 1), hi.cpu().reshape(-1, 1)
    outlier = (x < lo) | (x > hi)
    ptr = out["row_ptr"].cpu()
    assert torch.equal(ptr[1:] - ptr[:-1], outlier.sum(1)) and ptr[0] == 0
    n = int(ptr[-1])
    assert int(out["nnz"]) == n
    at = outlier.nonzero()
    assert torch.equal(out["col_idx"][:n].cpu().long(), at[:, 1])
    assert torch.equal(out["val"][:n].cpu(), (x - torch.where(x < lo, lo, hi))[outlier])
    assert torch.all(out["col_idx"][n:] == guard) and torch.all(out["val"][n:] == float(guard))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
# one wave a row, the workgroup, streamed rows (per tensor); rows of whole units of eight and others
@pytest.mark.parametrize("rows,cols,scope", [(r, c, s) for s in ("tensor", "token") for r, c in
                                             ((64, 96), (33, 1000), (16, 4096), (16, 4104), (8, 11008), (8, 16392), (5, 50))
                                             if s == "tensor" or c <= 16384])
@pytest.mark.parametrize("share", [0.004, 0.3])   # fewer than a tail holds; thresholds that are NaN themselves
def test_entries_are_what_was_counted(rows, cols, dtype, share, scope):
    from paper_2501_17116_amd import binding as b
    g = torch.Generator().manual_seed(rows + cols)
    x = torch.randn(rows, cols, generator=g)
    x[torch.rand(rows, cols, generator=g) < share] = float("nan")
    x[-1, -max(2, int(cols * share)):] = float("nan")     # the last segment ends where the entries end
    x = x.to(dtype)
    bits = x.view(torch.int16 if dtype == torch.bfloat16 else torch.int32)   # NaNs of either sign: at both ends of the order
    bits[x.isnan() & (torch.rand(rows, cols, generator=g) < 0.5)] |= torch.iinfo(bits.dtype).min
    x = x.cuda()
    alpha, guard = 0.95, -7
    L, ld = b.lib(), (cols + 7) // 8 * 8
    xp = torch.zeros(rows, ld, dtype=dtype, device="cuda")
    xp[:, :cols] = x
    token = scope == "token"
    cap = int(L.fp4_occ_capacity_token(rows, cols, alpha)) if token else b.occ_capacity(rows, cols, alpha)
    out = {"thresholds": torch.empty(2 * rows if token else 2, device="cuda"), "row_ptr": torch.empty(rows + 1, dtype=torch.int64, device="cuda"),
           "col_idx": torch.full((cap + 4096,), guard, dtype=torch.int32, device="cuda"), "val": torch.full((cap + 4096,), float(guard), device="cuda"),
           "nnz": torch.zeros(1, dtype=torch.int64, device="cuda")}
    ws = torch.empty(b.workspace_bytes(b.FP4_OP_OCC, rows, cols, 0, b._dt(x)), dtype=torch.uint8, device="cuda")
    fn = L.occ_clamp_residual_token if token else L.occ_clamp_residual
    assert fn(b._ptr(xp), b._dt(x), rows, cols, ld, alpha, b._ptr(out["thresholds"]), None, None, None, b._ptr(out["row_ptr"]), b._ptr(out["col_idx"]),
              b._ptr(out["val"]), cap, b._ptr(out["nnz"]), b._ptr(ws), ws.numel(), b._stream()) == 0
    thr = out["thresholds"].view(-1, 2)
    _check(out, x, thr[:, 0], thr[:, 1], guard)
