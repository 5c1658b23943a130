"""The rule that cuts an FP4 GEMM into tiles (csrc/gemm_tiling.h), on the CPU."""
import itertools

import pytest

from paper_2501_17116_amd import binding as b

LIMIT = 0xF0000000   # the staged tilings' offsets are 32 bits, and what they blank lies from here on


@pytest.mark.parametrize("row_bytes", [15_728_640, 15_728_656, 16_777_216, 31_457_280, 31_457_296, 33_554_432, 1 << 30])
def test_rows_stay_within_the_offsets(row_bytes):
    """Whatever the output's size and type, a staged tile's rows can be addressed."""
    for P, Q in itertools.product((64, 256, 4096, 40000), (64, 2048, 40000)):
        for factor, w_bf16, addend, out_bf16 in itertools.product((0, 1), repeat=4):
            tile, last_round = b.fp4_gemm_tiling(P, Q, 2 * row_bytes, factor, w_bf16, addend, out_bf16)
            assert tile == 64 or row_bytes * tile <= LIMIT, (P, Q, tile)
            assert last_round == 0 or tile == 256


@pytest.mark.parametrize("P,Q", [(1, 8), (4096, 4096), (40000, 40000)])
def test_an_empty_contraction_runs_where_nothing_is_requested_ahead(P, Q):
    for factor, w_bf16, addend, out_bf16 in itertools.product((0, 1), repeat=4):
        assert b.fp4_gemm_tiling(P, Q, 0, factor, w_bf16, addend, out_bf16) == (64, 0)
