"""Where the scales of a column-wise quantization are formed (csrc/quantize.hip), on the CPU."""
import pytest

from paper_2501_17116_amd import binding as b


@pytest.mark.parametrize("rows,cols,folds", [
    (8, 8, True), (512, 512, True), (2048, 2048, True), (8192, 2048, True), (4096, 4096, True), (65536, 256, True), (1024, 13824, True),
    (12288, 2048, True), (12544, 2048, False), (6144, 4096, True), (6144, 4160, False), (20000, 1024, True), (32768, 1024, True), (32768, 1032, False), (8192, 4096, False), (12288, 4096, False), (8192, 8192, False), (10208, 8256, False), (13824, 5120, False),
    (2048, 2050, False),       # rows of partial maxima that are not whole 16-byte words
    (131072, 64, True), (131072, 72, False),   # 128 MiB of partial maxima read by all tiles, and more
])
def test_lines(rows, cols, folds):
    assert b.fp4_quantize_cols_folds(rows, cols) == folds
