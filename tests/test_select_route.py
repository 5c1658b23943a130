"""Which passes find the clamp's thresholds (csrc/occ.hip), on the CPU."""
import pytest

from paper_2501_17116_amd import binding as b

BF16, F32 = b.FP4_BF16, b.FP4_F32


@pytest.mark.parametrize("rows,cols,windows", [
    (64, 2048, True), (64, 2056, False), (1056, 1376, True), (2049, 1032, True), (8192, 2048, True), (1024, 28672, True), (512, 13824, True),
    (256, 8192, True), (504, 504, True), (16, 504, True),
    # few long rows: a wave a row would leave most of the chip idle
    (1, 504, False), (1, 16384, False), (16, 16384, False), (32, 28672, False), (64, 13824, False), (128, 13824, False), (256, 13824, False),
    (480, 65504, False),
    # rows whose bins have no room, or that are not whole 16-byte words
    (8192, 496, False), (8192, 64, False), (8192, 508, False),
])
def test_windows_behind_a_digit(rows, cols, windows):
    assert b.fp4_select_route(rows, cols, BF16) & 3 == (b.FP4_SELECT_WINDOWS if windows else 0)
    assert b.fp4_select_route(rows, cols, F32) & 3 == 0
    assert b.fp4_select_route(rows, cols, BF16, ld=cols + 8) & 3 == 0


@pytest.mark.parametrize("rows,cols", [(16384, 4096), (16384, 11008), (4096, 8192), (1024, 65504), (66600, 504)])
def test_windows_behind_a_sample(rows, cols):
    assert b.fp4_select_route(rows, cols, BF16) & 3 == b.FP4_SELECT_WINDOWS | b.FP4_SELECT_SAMPLE


@pytest.mark.parametrize("rows,cols,found", [(64, 64, False), (65, 64, True), (64, 13824, False), (128, 13824, True), (4096, 64, True), (8192, 256, True),
                                             (262144, 32, True), (8192, 2048, False), (16384, 4096, False)])
def test_thresholds_in_a_launch_of_their_own(rows, cols, found):
    """Where more than a few workgroups count the rows behind a bf16 tensor's second digit."""
    assert bool(b.fp4_select_route(rows, cols, BF16) & b.FP4_SELECT_FOUND) == found
    if rows <= 65536:
        assert not b.fp4_select_route(rows, cols, F32) & b.FP4_SELECT_FOUND


@pytest.mark.parametrize("dt", [BF16, F32])
def test_rows_counted_by_themselves(dt):
    """Where the emitting kernel has no use for sums of blocks of rows, the count does not take eight rows a wave for them."""
    both = b.FP4_SELECT_FOUND | b.FP4_SELECT_APART
    for rows, cols in ((65537, 64), (131072, 32), (262144, 256)):
        assert b.fp4_select_route(rows, cols, dt) == both
    assert not b.fp4_select_route(65536, 64, dt) & b.FP4_SELECT_APART
