"""What a layer's launches do beside their own work, on either side of each line (csrc/quantize.hip), on the CPU."""
import pytest

from paper_2501_17116_amd import binding as b

BF16, F32 = b.FP4_BF16, b.FP4_F32


@pytest.mark.parametrize("M,K,N,dt,want", [
    # bf16: one tile a workgroup, up to 1024 of them (K 256 by N 64), or apart; beyond some tokens a sample takes the digits' place
    (32, 2048, 5504, BF16, 1), (64, 4096, 4096, BF16, 1), (64, 4096, 4160, BF16, 0), (32, 4096, 8192, BF16, 0),
    # fp32: two rounds of workgroups, with one or two tiles each
    (256, 512, 512, F32, 1), (2048, 2048, 2048, F32, 1), (2304, 2048, 2080, F32, 2), (4096, 2048, 4096, F32, 2), (1024, 4096, 2048, F32, 2),
    # with four: where the digit pass leaves CUs, or the tiles are a round of their own
    (256, 2048, 8192, F32, 4), (512, 3072, 4096, F32, 4), (4096, 4096, 4096, F32, 4), (1024, 3072, 4096, F32, 0), (2048, 4096, 3072, F32, 0),
    (2048, 2048, 5504, F32, 0), (256, 8192, 4096, F32, 0),
])
def test_digit_pass_beside_the_weights(M, K, N, dt, want):
    assert b.fp4_select_beside(M, K, N, dt) == want


@pytest.mark.parametrize("M,K,N,want", [
    (32, 32, 32, 1), (1536, 2048, 2048, 1), (2048, 2048, 2048, 2), (4096, 2048, 2048, 4), (1024, 8192, 2048, 2), (8192, 1024, 2048, 4),
    (8192, 1024, 2304, 0), (8192, 2048, 2048, 0), (16384, 512, 512, 4), (16640, 512, 512, 0), (64, 8192, 64, 1), (64, 8224, 64, 0),
])
def test_transposition_beside_the_codes(M, K, N, want):
    assert b.fp4_transpose_beside(M, K, N) == want


@pytest.mark.parametrize("M,K,N,alpha,bf16,f32", [
    (256, 512, 512, 0.99, 1, 1), (512, 2048, 512, 0.99, 1, 1), (64, 3072, 2048, 0.999, 1, 1), (1024, 1024, 1024, 0.97, 1, 0),
    # more entries in 64 rows than 256 threads count while the others run: later beside wide rows of bf16
    (512, 1376, 2048, 0.97, 0, 0), (64, 2048, 2048, 0.97, 0, 0), (512, 4096, 512, 0.99, 0, 0), (64, 3072, 5504, 0.985, 1, 0), (64, 3072, 5504, 0.97, 0, 0),
    (32, 1376, 11008, 0.9, 0, 0), (48, 96, 96, 0.9, 1, 1),
    # more than four workgroups a CU; columns beyond the masks
    (8192, 512, 512, 0.99, 0, 0), (64, 4128, 64, 0.999, 0, 0),
])
def test_count_beside_the_rows(M, K, N, alpha, bf16, f32):
    cap = b.occ_capacity(M, K, alpha)
    assert b.fp4_count_beside(M, K, N, BF16, cap) == bool(bf16) and b.fp4_count_beside(M, K, N, F32, cap) == bool(f32)


def test_count_beside_with_cached_weights_and_any_capacity():
    assert not b.fp4_count_beside(64, 4096, 64, BF16, 64)          # 1024 workgroups have W's rows
    assert b.fp4_count_beside(64, 4096, 64, BF16, 64, cached=True)
    assert not b.fp4_count_beside(64, 1024, 64, BF16, 2 ** 62)     # as many as are provided for
