"""No-GPU checks of the boundary: the library loads, exports every declared symbol, validates
arguments before launching anything, and its rounding routine (run on the host) agrees with
the oracle bit for bit."""
import ctypes as C
import itertools
import os
import re

import numpy as np
import pytest

from oracle import fp4_oracle as o
from paper_2501_17116_amd import binding as b

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(b.LIB_PATH):
        pytest.fail("libfp4mi.so is not built; run __graft_entry__.build() first")
    return b.lib()


def _declared_symbols():
    src = "".join(open(os.path.join(ROOT, "include", h)).read()
                  for h in sorted(os.listdir(os.path.join(ROOT, "include"))) if h.endswith(".h"))
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    names = re.findall(r"\b(?:int|size_t|int64_t|const char\*)\s+(\w+)\s*\(", src)
    return sorted(set(names))


def test_every_declared_symbol_is_exported(L):
    names = _declared_symbols()
    for must in ("fp4_quantize", "occ_clamp_residual", "fp4_linear_fwd", "fp4_linear_bwd_dgrad",
                 "fp4_linear_bwd_wgrad"):
        assert must in names
    for n in names:
        assert hasattr(L, n), n


def test_status_strings_and_queries(L):
    assert b.status_string(0) == "ok"
    assert "shape" in b.status_string(-2)
    assert b.occ_capacity(256, 512, 0.99) == 2 * o.occ_tail_count(256 * 512, 0.99) == 2620
    assert b.occ_capacity(16384, 4096, 0.999) == 2 * o.occ_tail_count(16384 * 4096, 0.999)
    assert b.occ_capacity(4, 4, 1.0) == 0
    assert b.occ_capacity(4, 4, 0.3) == -1
    for op in range(9):
        assert b.workspace_bytes(op, 256, 512, 512, b.FP4_F32) > 0
    # the one-call backward needs at least what either gradient needs alone
    for dt in (b.FP4_F32, b.FP4_BF16):
        both = b.workspace_bytes(b.FP4_OP_BWD, 256, 512, 512, dt)
        assert both >= b.workspace_bytes(b.FP4_OP_DGRAD, 256, 512, 512, dt)
        assert both >= b.workspace_bytes(b.FP4_OP_WGRAD, 256, 512, 512, dt)
    assert L.fp4_occ_capacity_token(100, 1000, 0.99) == 100 * 2 * o.occ_tail_count(1000, 0.99) == 2000
    assert L.fp4_occ_capacity_token(4, 8, 1.0) == 0 and L.fp4_occ_capacity_token(4, 8, 0.2) == -1
    assert b.workspace_bytes(99, 256, 512, 512, b.FP4_F32) == 0
    # forward workspace holds at least both packed operands and the fp32 residual product
    M, K, N = 16384, 4096, 12288
    assert b.workspace_bytes(b.FP4_OP_FWD, M, K, N, b.FP4_BF16) >= M * K // 2 + N * K // 2 + 4 * M * N


def test_argument_validation_happens_on_the_host(L):
    one = C.c_void_p(16)   # non-null, aligned, never dereferenced: every call below must fail first
    assert L.fp4_quantize(None, 0, 4, 8, 8, 0, one, one, one, 1 << 20, None) == -1
    assert L.fp4_quantize(one, 0, 4, 7, 8, 0, one, one, one, 1 << 20, None) == -2      # odd cols
    assert L.fp4_quantize(one, 7, 4, 8, 8, 0, one, one, one, 1 << 20, None) == -3
    assert L.fp4_quantize(one, 0, 4, 8, 4, 0, one, one, one, 1 << 20, None) == -2      # ld < cols
    assert L.fp4_quantize(C.c_void_p(20), 0, 4, 8, 8, 0, one, one, one, 1 << 20, None) == -4
    assert L.fp4_quantize(one, 0, 4, 8, 8, 1, one, one, None, 0, None) == -5            # col needs ws
    assert L.fp4_quantize(one, 0, 0, 8, 8, 0, one, one, one, 0, None) == 0              # empty: no-op
    assert L.fp4_gemm(one, one, one, one, 4, 4, 48, None, one, 0, 8, None) == -2        # K % 32
    assert L.fp4_gemm(one, None, one, None, 4, 4, 64, None, one, 1, 8, None) == -3      # raw needs fp32
    assert L.fp4_gemm(one, one, one, one, 0, 4, 64, None, one, 0, 8, None) == 0
    ctx = b.fp4_fwd_ctx(16, 16, 16, 16, 16, 0, 16)
    big = 1 << 40
    assert L.fp4_linear_fwd(one, one, 0, 8, 48, 8, 0.99, one, C.byref(ctx), one, big, None) == -2
    assert L.fp4_linear_fwd(one, one, 0, 8, 64, 8, 0.2, one, C.byref(ctx), one, big, None) == -4
    assert L.fp4_linear_fwd(one, one, 0, 8, 64, 8, 0.99, one, C.byref(ctx), one, big, None) == -6  # capacity 0 < 2k
    assert L.fp4_linear_fwd(one, one, 0, 8, 64, 8, 1.0, one, C.byref(ctx), one, 8, None) == -5
    assert L.fp4_linear_bwd_dgrad(one, one, 0, 8, 8, 48, one, one, big, None) == -2
    assert L.fp4_linear_bwd_wgrad(one, one, one, 0, 48, 8, 8, C.byref(ctx), 5.0, 3.0, one, one, big, None) == -2
    assert L.fp4_linear_bwd_wgrad(one, one, one, 0, 64, 8, 8, C.byref(ctx), 5.0, -1.0, one, one, big, None) == -4
    assert L.occ_clamp_residual(one, 0, 8, 8, 8, 0.9, one, None, None, None, one, one, one, 0, one, one, big,
                                None) == -6
    assert L.fp4_dge_apply(one, one, 0, one, 8, 12, 5.0, 3.0, one, None) == -2


def test_argument_validation_of_the_wider_entry_points(L):
    # same rule: every call fails on the host, before anything could be enqueued
    one = C.c_void_p(16)
    big = 1 << 40
    roomy = b.fp4_fwd_ctx(16, 16, 16, 16, 16, 1 << 30, 16, b.FP4_OCC_TENSOR)
    token = b.fp4_fwd_ctx(16, 16, 16, 16, 16, 1 << 30, 16, b.FP4_OCC_TOKEN)
    noscope = b.fp4_fwd_ctx(16, 16, 16, 16, 16, 1 << 30, 16, 5)
    wq = b.fp4_weight_cache(16, 16, 16, 16)
    holed = b.fp4_weight_cache(16, 16, 0, 16)
    bwd = lambda dY, wqp, M, N, ctx, cap, ws: L.fp4_linear_bwd(dY, one, one, wqp, 0, M, 64, N, C.byref(ctx), 5.0, cap,
                                                               one, one, one, ws, None)
    assert bwd(None, None, 64, 64, roomy, 3.0, big) == -1
    assert bwd(one, None, 48, 64, roomy, 3.0, big) == -2             # tokens are contracted: M % 32
    assert bwd(one, None, 64, 48, roomy, 3.0, big) == -2             # output channels are contracted: N % 32
    assert bwd(one, None, 64, 64, roomy, 0.0, big) == -4             # cap <= 0
    assert bwd(one, None, 64, 64, roomy, 3.0, 8) == -5
    assert bwd(one, None, 64, 64, noscope, 3.0, big) == -3
    assert bwd(one, C.byref(holed), 64, 64, roomy, 3.0, big) == -1
    assert L.fp4_prepare_weights(one, 0, 48, 64, C.byref(wq), one, big, None) == -2
    assert L.fp4_prepare_weights(one, 0, 64, 64, C.byref(holed), one, big, None) == -1
    assert L.fp4_prepare_weights(one, 0, 64, 64, C.byref(wq), one, 8, None) == -5
    assert L.fp4_linear_fwd_cached(one, one, None, 0, 8, 64, 64, 0.99, one, C.byref(roomy), one, big, None) == -1
    assert L.fp4_linear_fwd_cached(one, one, C.byref(wq), 0, 8, 48, 64, 0.99, one, C.byref(roomy), one, big, None) == -2
    assert L.fp4_linear_bwd_dgrad_cached(one, C.byref(wq), 0, 8, 64, 48, one, one, big, None) == -2
    assert L.fp4_linear_bwd_dgrad_cached(one, None, 0, 8, 64, 64, one, one, big, None) == -1
    # per-token thresholds: rows have to fit the registers of a workgroup
    tok = lambda cols, alpha, cap: L.occ_clamp_residual_token(one, 0, 8, cols, cols, alpha, one, None, None, None, one,
                                                              one, one, cap, one, one, big, None)
    assert tok(16392, 0.99, big) == -2
    assert tok(64, 0.9, 0) == -6
    assert tok(64, 0.7, big) == -4
    assert L.fp4_linear_fwd(one, one, 0, 8, 16416, 8, 0.99, one, C.byref(token), one, big, None) == -2
    assert L.fp4_linear_fwd(one, one, 0, 8, 64, 8, 0.99, one, C.byref(noscope), one, big, None) == -3
    # FP8 quantizer and the mixed-format calls
    assert L.fp8_quantize(None, 0, 4, 8, 8, 0, one, one, one, big, None) == -1
    assert L.fp8_quantize(one, 0, 4, 8, 4, 0, one, one, one, big, None) == -2
    assert L.fp8_quantize(one, 9, 4, 8, 8, 0, one, one, one, big, None) == -3
    assert L.fp8_quantize(one, 0, 4, 8, 8, 1, one, one, None, 0, None) == -5
    assert L.fp8_quantize(one, 0, 0, 8, 8, 0, one, one, one, 0, None) == 0
    mixed = lambda fl, fr, P, Kc: L.fp4_gemm_mixed(one, fl, one, one, fr, one, P, 4, Kc, None, one, 0, 8, None)
    assert mixed(b.FP4_FMT_E2M1, b.FP4_FMT_E2M1, 4, 128) == -3      # exactly one operand is 8-bit
    assert mixed(b.FP4_FMT_E4M3, b.FP4_FMT_E4M3, 4, 128) == -3
    assert mixed(3, b.FP4_FMT_E2M1, 4, 128) == -3
    assert mixed(b.FP4_FMT_E4M3, b.FP4_FMT_E2M1, 4, 64) == -2       # K % 128
    assert mixed(b.FP4_FMT_E4M3, b.FP4_FMT_E2M1, 0, 128) == 0
    fwdm = lambda K, fa, fw, alpha, ws: L.fp4_linear_fwd_mixed(one, one, 0, 8, K, 8, fa, fw, alpha, one,
                                                               C.byref(roomy), one, ws, None)
    assert fwdm(128, b.FP4_FMT_E4M3, b.FP4_FMT_E2M1, 0.99, big) == -4   # FP8 activations run without the clamp
    assert fwdm(64, b.FP4_FMT_E4M3, b.FP4_FMT_E2M1, 1.0, big) == -2
    assert fwdm(128, b.FP4_FMT_E2M1, b.FP4_FMT_E2M1, 1.0, big) == -3
    assert fwdm(128, b.FP4_FMT_E4M3, b.FP4_FMT_E2M1, 1.0, 8) == -5
    # tensor-wise scaling: an axis of fp4_quantize and a forward pass of its own
    assert L.fp4_quantize(one, 0, 4, 7, 8, b.FP4_AXIS_TENSOR, one, one, one, 1 << 20, None) == -2     # odd cols
    assert L.fp4_quantize(one, 0, 4, 8, 8, b.FP4_AXIS_TENSOR, one, one, None, 0, None) == -5          # needs a workspace
    assert L.fp4_quantize(one, 0, 4, 8, 8, 3, one, one, one, 1 << 20, None) == -3
    gran = lambda K, a_t, w_t, alpha, ctx, ws: L.fp4_linear_fwd_granularity(one, one, 0, 8, K, 8, a_t, w_t, alpha, one,
                                                                           C.byref(ctx), one, ws, None)
    assert gran(48, 1, 0, 0.99, roomy, big) == -2
    assert gran(64, 1, 0, 0.2, roomy, big) == -4
    assert gran(64, 1, 0, 0.99, token, big) == -4        # per-token thresholds with one scale per tensor
    assert gran(64, 1, 1, 0.99, roomy, 8) == -5
    # the entry point that allocates nothing refuses what its built-in scratch cannot hold
    assert L.fp4_quantize_noalloc(None, 0, 4, 8, 8, 0, one, one, None) == -1
    assert L.fp4_quantize_noalloc(one, 0, 4, 7, 8, 0, one, one, None) == -2
    assert L.fp4_quantize_noalloc(one, 1, 1 << 20, 16384, 16384, 1, one, one, None) == -8
    assert L.fp4_quantize_noalloc(one, 0, 0, 8, 8, 0, one, one, None) == 0
    assert "scratch" in b.status_string(-8) or "limit" in b.status_string(-8)


def test_library_rounding_equals_the_oracle_bit_for_bit(L):
    rng = np.random.default_rng(0)
    # every threshold and grid point with its fp32 neighbours, both signs, specials
    pts = [0.25, 0.5, 0.75, 1, 1.25, 1.5, 1.75, 2, 2.5, 3, 3.5, 4, 5, 6, 7, 0.0]
    edge = []
    for p in pts:
        for s in (1, -1):
            v = np.float32(s * p)
            edge += [v, np.nextafter(v, np.float32(np.inf)), np.nextafter(v, np.float32(-np.inf))]
    edge += [np.float32(x) for x in (np.inf, -np.inf, np.nan, 1e-45, -1e-45, 1e38, -1e38, -0.0)]
    edge = np.array(edge, np.float32)
    assert np.array_equal(b.fp4_host_round_codes(edge), o.q_e2m1(edge))
    # random bit patterns (all exponents) and a dense sweep of the interesting range
    bits = rng.integers(0, 2 ** 32, 4_000_000, dtype=np.uint64).astype(np.uint32)
    x = bits.view(np.float32)
    assert np.array_equal(b.fp4_host_round_codes(x), o.q_e2m1(x))
    x = rng.uniform(-7, 7, 4_000_000).astype(np.float32)
    assert np.array_equal(b.fp4_host_round_codes(x), o.q_e2m1(x))
    # the mantissa patterns around every tie, in every binade the grid spans
    base = np.array([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0], np.float32).view(np.uint32)
    near = (base[:, None].astype(np.int64) + np.arange(-2000, 2001)[None, :]).astype(np.uint32).ravel()
    for sign in (0, 0x80000000):
        x = (near | np.uint32(sign)).view(np.float32)
        assert np.array_equal(b.fp4_host_round_codes(x), o.q_e2m1(x))


def test_library_fp8_rounding_equals_the_oracle_bit_for_bit(L):
    rng = np.random.default_rng(1)
    grid = o.e4m3_decode(np.arange(0x7F, dtype=np.uint8)).astype(np.float64)
    mids = ((grid[:-1] + grid[1:]) / 2).astype(np.float32)
    edge = np.concatenate([grid.astype(np.float32), mids, np.nextafter(mids, np.float32(np.inf)),
                           np.nextafter(mids, np.float32(-np.inf)),
                           np.array([0.0, -0.0, 448, 449, 464, 480, 1e9, 1e-45, 2.0 ** -10, 2.0 ** -9 * 7.5], np.float32)])
    edge = np.concatenate([edge, -edge])
    assert np.array_equal(b.fp8_host_round_codes(edge), o.q_e4m3(edge))
    for x in (rng.uniform(-460, 460, 2_000_000), rng.normal(size=2_000_000) * 0.02,
              np.exp(rng.uniform(-25, 8, 2_000_000)) * rng.choice([-1, 1], 2_000_000)):
        x = x.astype(np.float32)
        assert np.array_equal(b.fp8_host_round_codes(x), o.q_e4m3(x))


def test_a_smaller_problem_never_needs_a_larger_workspace(L):
    """A buffer sized for the largest shape serves every smaller one, across the sizes at which a kernel changes its block,
    slice or path."""
    rng = np.random.default_rng(5)
    edges = [64, 512, 1024, 2048, 4096, 7136, 8064, 8160, 8192, 8224, 11008, 12288, 16288, 16384, 24576, 24608, 32768]

    def size():
        return int(rng.choice(edges)) if rng.random() < 0.5 else 32 * int(np.exp(rng.uniform(np.log(1), np.log(1024))))

    def bytes_of(op, s, dt):
        return b.workspace_bytes(op, *s, dt)

    for op in range(9):
        for dt in (b.FP4_F32, b.FP4_BF16):
            assert bytes_of(op, (8064, 2048, 2048), dt) <= bytes_of(op, (8192, 2048, 2048), dt)
            assert bytes_of(op, (16288, 11008, 4096), dt) <= bytes_of(op, (16384, 11008, 12288), dt)
            for _ in range(3000):
                big = (size(), size(), size())
                small = tuple(min(x, size()) if rng.random() < 0.6 else x for x in big)
                assert bytes_of(op, small, dt) <= bytes_of(op, big, dt), (op, dt, small, big)


@pytest.mark.parametrize("op", range(9))
def test_workspaces_grow_along_every_dimension(L, op):
    """Each dimension by itself, in the smallest steps, past every size at which a path begins or ends; the other two at
    sizes on either side of those."""
    around = [v + d for v in (64, 512, 1024, 2048, 4096, 8192, 16384, 24576, 32768, 65536) for d in (-32, 0, 32)]
    for dt in (b.FP4_F32, b.FP4_BF16):
        for dim in range(3):
            for other in itertools.product((32, 4096, 8224, 16384, 65536), repeat=2):
                need = [b.workspace_bytes(op, *other[:dim], v, *other[dim:], dt) for v in around]
                for v, less, more in zip(around[1:], need, need[1:]):
                    assert less <= more, (dt, dim, other, v)


def test_residual_temporaries_and_product_share_their_room(L):
    """Forward and weight gradient hold either the unordered entries or the product's scratch at a time."""
    MiB = 1 << 20
    for M, K, N in ((16384, 11008, 4096), (16384, 4096, 12288), (4096, 5120, 13824)):
        entries = 8 * b.occ_capacity(M, K, 0.9)
        codes = (M + N) * K // 2
        fwd = b.workspace_bytes(b.FP4_OP_FWD, M, K, N, b.FP4_BF16)
        assert fwd <= codes + 4 * M * N + max(entries, b.workspace_bytes(b.FP4_OP_SPMM, M, K, N, b.FP4_BF16)) + 4 * MiB
        wgrad = b.workspace_bytes(b.FP4_OP_WGRAD, M, K, N, b.FP4_BF16)
        masks = 8 * ((M + 63) // 64) * K   # the transposition's counts and offsets
        assert wgrad <= (K + N) * M // 2 + entries + max(entries + masks, b.workspace_bytes(b.FP4_OP_SPMM, K, M, N, b.FP4_BF16)) + 12 * MiB
