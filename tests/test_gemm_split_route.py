"""Where an FP4 GEMM takes the 32 x 32 tiles whose waves share a contraction (csrc/gemm_tiling.h), on the CPU."""
import pytest

from paper_2501_17116_amd import binding as b


@pytest.mark.parametrize("P,Q,Kc,factor,want", [
    (64, 2048, 512, 0, 1), (64, 2048, 256, 0, 0), (64, 2048, 1120, 0, 1), (64, 2048, 1088, 0, 0), (512, 512, 256, 1, 1), (512, 512, 224, 1, 0),
    # 512 tiles and more, 768 and more
    (512, 1024, 512, 0, 1), (512, 1056, 512, 0, 0), (512, 1056, 1024, 0, 1), (512, 1056, 3040, 0, 0), (512, 1056, 3104, 0, 1), (512, 1056, 4096, 1, 0),
    (768, 1024, 4096, 0, 1), (768, 1056, 4096, 0, 0), (1, 8, 0, 0, 0),
    # 36 a product: sums up to 2^22 are exact in fp32, in four chains as in one
    (32, 64, 116480, 0, 1), (32, 64, 116512, 0, 0), (512, 512, 116480, 1, 1), (512, 512, 116512, 1, 0), (32, 64, 2 * 0x7800000, 0, 0),
])
def test_lines(P, Q, Kc, factor, want):
    assert b.fp4_gemm_splits(P, Q, Kc, factor) == bool(want)
