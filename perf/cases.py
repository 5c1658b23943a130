"""What the FP4 linear layer is timed on: training steps, forward and backward passes of single layers.

A case is one layer (M tokens, K input channels, N output channels), a master data type, the clamp's
alpha and scope, and what of the layer runs: "step" (forward, then both gradients in one call),
"separate" (forward, activation gradient and weight gradient as three calls), "forward", "backward" (both
gradients from a saved forward context).  "cached" takes the weights' quantizations from a cache, as a
program does that runs several micro-batches between two optimizer steps.

The shapes are those of the benchmark's workloads (LLaMA-2 1.3B, 7B and 13B linear layers), of the tests,
and generic ones; the inputs follow the benchmark's recipe: weights N(0, 0.02^2), output gradients
N(0, 0.01^2), activations either N(0, 1) with a few channels scaled up or Student-t with three degrees of
freedom.
"""
import math

import torch

from paper_2501_17116_amd import binding as b

DGE_K, DGE_CAP = 5.0, 3.0


def _case(name, run, M, K, N, dtype="bf16", alpha=0.99, act="channels", scope="tensor", cached=False):
    return {"name": name, "run": run, "M": M, "K": K, "N": N, "dtype": dtype, "alpha": alpha, "act": act,
            "scope": scope, "cached": cached}


def listed():
    return [
        # the smallest configuration: one fp32 layer, where launches and host work count
        _case("fp32-256x512x512", "step", 256, 512, 512, dtype="f32"),
        # a short batch through a layer whose weights are quantized already: the latency of a forward pass
        _case("fwd-64x2048x2048-cached", "forward", 64, 2048, 2048, cached=True),
        # 1.3B-shaped layers: the square one, and the ragged width of the feed-forward layer with the three
        # passes called one by one
        _case("1.3B-o-8192x2048x2048", "step", 8192, 2048, 2048),
        _case("1.3B-gate-8192x2048x5504", "separate", 8192, 2048, 5504),
        # 7B-shaped layers: the largest training step; a micro-batch without the clamp on cached weights;
        # the long contraction of the down projection, forward only; the backward pass alone
        _case("7B-qkv-16384x4096x12288", "step", 16384, 4096, 12288),
        _case("7B-o-16384x4096x4096-noclamp", "step", 16384, 4096, 4096, alpha=1.0, cached=True),
        _case("7B-down-16384x11008x4096-fwd", "forward", 16384, 11008, 4096),
        _case("7B-gate-8192x4096x11008-bwd", "backward", 8192, 4096, 11008),
        # 13B-shaped layer, heavy-tailed activations, the lightest clamp in use
        _case("13B-ffn-4096x5120x13824-t3", "step", 4096, 5120, 13824, alpha=0.999, act="student-t"),
        # thresholds per token instead of per tensor
        _case("7B-gate-4096x4096x11008-token", "step", 4096, 4096, 11008, scope="token"),
        # no dimension a multiple of a tile, the densest residual in use
        _case("odd-1056x1376x2080", "step", 1056, 1376, 2080, alpha=0.97),
        # fp32 masters at an ordinary size
        _case("fp32-2048x2048x2048", "step", 2048, 2048, 2048, dtype="f32"),
    ]


def _density(alpha):
    return 2.0 * (1.0 - alpha)


def _cost(c):
    """Rough relative cost of a case: dense work, plus the residual's, which runs far from the matrix peak."""
    passes = {"step": 1.0, "separate": 1.0, "forward": 0.4, "backward": 0.7}[c["run"]]
    return passes * float(c["M"]) * c["K"] * c["N"] * (1.0 + 65.0 * _density(c["alpha"])) * (4.0 if c["dtype"] == "f32" else 1.0)


def draw(rng):
    """One more case of the same ranges; sizes over their logarithm, multiples of 32 (what the layer takes)."""
    def size(lo, hi):
        return max(lo, min(hi, 32 * round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 32)))

    most = max(_cost(c) for c in listed())
    while True:
        f32 = rng.random() < 0.2
        c = {
            "run": rng.choice(["step", "step", "step", "separate", "forward", "forward", "backward"]),
            "M": size(64, 4096 if f32 else 16384),
            "K": size(512, 4096 if f32 else 13824),
            "N": size(512, 4096 if f32 else 15360),
            "dtype": "f32" if f32 else "bf16",
            "alpha": rng.choice([0.99, 0.99, 0.99, 0.999, 0.97, 1.0]),
            "act": rng.choice(["channels", "channels", "student-t"]),
            "scope": "token" if rng.random() < 0.2 else "tensor",
            "cached": rng.random() < 0.3,
        }
        if _cost(c) <= most:
            return c


def prepare(case, seed):
    M, K, N = case["M"], case["K"], case["N"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + 17)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)

    A = normal(M, K)
    if case["act"] == "channels":
        frac, scale = (0.001, 50.0) if case["dtype"] == "bf16" else (0.005, 20.0)
        ch = torch.randperm(K, generator=g, device="cuda")[:max(1, round(frac * K))]
        A[:, ch] *= scale
    else:
        A /= torch.sqrt((normal(M, K) ** 2 + normal(M, K) ** 2 + normal(M, K) ** 2) / 3.0)
    scope = b.FP4_OCC_TOKEN if case["scope"] == "token" else b.FP4_OCC_TENSOR
    s = {"case": case, "A": A.to(dt), "W": (normal(K, N) * 0.02).to(dt), "wq": None,
         "ctx": b.FwdCtx(M, K, N, case["alpha"], scope=scope), "Y": torch.empty(M, N, device="cuda", dtype=dt)}
    if case["cached"]:
        s["wq"] = b.fp4_prepare_weights(s["W"])
    if case["run"] != "forward":
        s["dY"] = (normal(M, N) * 0.01).to(dt)
        s["dA"] = torch.empty(M, K, device="cuda", dtype=dt)
        s["dW"] = torch.empty(K, N, device="cuda", dtype=torch.float32)
    if case["run"] == "backward":
        _forward(s)
    return s


def _forward(s):
    if s["wq"] is not None:
        b.fp4_linear_fwd_cached(s["A"], s["W"], s["wq"], s["case"]["alpha"], ctx=s["ctx"], Y=s["Y"])
    else:
        b.fp4_linear_fwd(s["A"], s["W"], s["case"]["alpha"], ctx=s["ctx"], Y=s["Y"])


def run(state):
    s, ctx = state, state["ctx"]
    what = s["case"]["run"]
    out = {}
    if what != "backward":
        _forward(s)
        out.update(Y=s["Y"], gamma_W=ctx.gamma_W)
        if s["case"]["alpha"] < 1.0:
            out.update(thresholds=ctx.thresholds, row_ptr=ctx.row_ptr, nnz=ctx.nnz)
    if what == "separate":
        if s["wq"] is not None:
            b.fp4_linear_bwd_dgrad_cached(s["dY"], s["wq"], dA=s["dA"])
        else:
            b.fp4_linear_bwd_dgrad(s["dY"], s["W"], dA=s["dA"])
        b.fp4_linear_bwd_wgrad(s["A"], s["dY"], s["W"], ctx, DGE_K, DGE_CAP, dW=s["dW"])
    elif what != "forward":
        b.fp4_linear_bwd(s["dY"], s["A"], s["W"], ctx, DGE_K, DGE_CAP, wq=s["wq"], dA=s["dA"], dW=s["dW"])
    if what != "forward":
        out.update(dA=s["dA"], dW=s["dW"])
    return out


def work(case):
    """Inputs once, outputs once, the residual's entries once each way they go; products without padding."""
    M, K, N = case["M"], case["K"], case["N"]
    e = 2 if case["dtype"] == "bf16" else 4
    nnz = _density(case["alpha"]) * M * K
    entries = 8.0 * nnz + 8.0 * (M + 1)
    products = {"forward": 1, "backward": 2}.get(case["run"], 3)
    residuals = {"forward": 1, "backward": 1}.get(case["run"], 2)
    size = float(M * K + K * N) * e                                   # A, W
    if case["run"] != "backward":
        size += M * N * e + 4.0 * N + entries                         # Y, scales, residual out
    if case["cached"]:
        size += K * N * (0.5 if case["run"] in ("forward", "backward") else 1.0)
    if case["run"] != "forward":
        size += M * N * e + M * K * e + 4.0 * K * N                   # dY; dA, dW out
        if case["run"] == "backward":
            size += entries
    return {"bytes": size, "flops": 2.0 * products * M * K * N + 2.0 * residuals * nnz * N}


def tolerance(case):
    """About four times what separates the outputs from an fp64 evaluation of the same codes, scales, thresholds
    and residual, rounded to the output type: bf16 outputs 8e-5 (values on the verge of a rounding that go to the
    neighbour) and 7e-3 for a single value (one bf16 step); fp32 outputs 6e-7 and 4e-5 (the weight gradient's
    derivative factor next to its pole).  Thresholds, scales and row pointers come out the same."""
    return {"rel": 3e-4, "max": 0.03} if case["dtype"] == "bf16" else {"rel": 2.5e-6, "max": 2e-4}


# The layer once more, from its definition and in plain torch: what decides a code, a threshold or a residual
# entry in fp32 (as the layer defines it), the products and everything behind them in fp64.

def _codes(x, dim):
    """E2M1 values (fp64) and fp32 scales of x [..] under one scale 6 / absmax along dim; midpoints go up."""
    top = x.abs().amax(dim=dim, keepdim=True)
    gamma = (6.0 / top.double()).float()   # the correctly rounded quotient: a code on a midpoint hangs on its last bit
    gamma = torch.where((top > 0) & torch.isfinite(gamma), gamma, torch.ones_like(gamma))
    pos = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]
    grid = torch.tensor([-v for v in pos[:0:-1]] + pos, device=x.device)
    mid = (grid[1:] + grid[:-1]) / 2
    return grid.double()[torch.bucketize(x * gamma, mid, right=True)], gamma


def exact(case, seed):
    s = prepare(dict(case, run="step", cached=False), seed)
    A, W, dY = s["A"].float(), s["W"].float(), s["dY"].float()
    M, K = A.shape
    out = {}
    qW, gW = _codes(W, 0)
    rest = None
    if case["alpha"] < 1.0:
        token = case["scope"] == "token"
        flat = (A if token else A.reshape(1, -1)).sort(dim=1).values
        k = math.floor((1.0 - case["alpha"]) * flat.shape[1])
        lo, hi = flat[:, k:k + 1], flat[:, flat.shape[1] - 1 - k:flat.shape[1] - k]
        del flat
        Ac = torch.minimum(torch.maximum(A, lo), hi)
        rest = A - Ac
        per_row = (rest != 0).sum(dim=1)
        row_ptr = torch.zeros(M + 1, dtype=torch.int64, device=A.device)
        torch.cumsum(per_row, 0, out=row_ptr[1:])
        rest = rest.double()
    else:
        Ac = A
    if case["run"] != "backward":
        qA, gA = _codes(Ac, 1)
        Y = (qA @ qW) / (gA.double() * gW.double())
        if rest is not None:
            Y += rest @ W.double()
        out.update(Y=Y, gamma_W=gW.reshape(-1))
        if rest is not None:
            out.update(thresholds=torch.cat([lo, hi], dim=1).reshape(s["ctx"].thresholds.shape), row_ptr=row_ptr,
                       nnz=row_ptr[-1:].reshape(s["ctx"].nnz.shape))
    if case["run"] != "forward":
        qY, gY = _codes(dY, 1)
        qR, gR = _codes(W, 1)
        out["dA"] = (qY @ qR.t()) / (gY.double() * gR.reshape(1, -1).double())
        qC, gC = _codes(Ac, 0)
        qD, gD = _codes(dY, 0)
        dW = (qC.t() @ qD) / (gC.reshape(-1, 1).double() * gD.double())
        if rest is not None:
            dW += rest.t() @ dY.double()
        a = (W * gW).abs()
        left = torch.where(a >= 4, 4.0, torch.where(a >= 2, a.floor(), (2 * a).floor() / 2)).double()
        width = torch.where(a >= 4, 2.0, torch.where(a >= 2, 1.0, 0.5)).double()
        t = (2.0 * (a.double() - left) / width - 1.0).abs()
        out["dW"] = dW * torch.clamp(t ** (1.0 / DGE_K - 1.0) / DGE_K, max=DGE_CAP)
    return out
