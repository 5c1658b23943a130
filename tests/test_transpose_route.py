"""Where the places of the transposed residual's entries come from (csrc/spmm.hip), on the CPU."""
import pytest

from paper_2501_17116_amd import binding as b

FEW, SCAN, TABLE = 1, 2, 3


@pytest.mark.parametrize("P,Q,want", [
    (32, 64, FEW), (256, 512, FEW), (1056, 1376, FEW), (1024, 4096, FEW), (1088, 4096, SCAN), (512, 8192, FEW), (576, 8192, SCAN),
    (96, 16384, FEW), (160, 16384, SCAN), (4096, 1024, FEW), (4128, 992, SCAN),
    # counts of few columns, but of so many blocks that adding them up in every workgroup takes longer than a launch
    (8192, 128, SCAN), (16384, 128, SCAN), (65536, 64, SCAN), (131072, 32, SCAN),
    # positions of 32 bits
    (262144, 16352, SCAN), (262144, 16384, TABLE), (1 << 20, 4096, TABLE), ((1 << 20) - 32, 4096, SCAN),
    (32, 16416, 0),
])
def test_lines(P, Q, want):
    assert b.fp4_residual_transpose_positions(P, Q) == want
