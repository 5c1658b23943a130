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
            tile, last_round, _ = b.fp4_gemm_tiling(P, Q, 2 * row_bytes, factor, w_bf16, addend, out_bf16)
            assert tile == 64 or row_bytes * tile <= LIMIT, (P, Q, tile)
            assert last_round == 0 or tile == 256


@pytest.mark.parametrize("P,Q", [(1, 8), (4096, 4096), (40000, 40000)])
def test_an_empty_contraction_runs_where_nothing_is_requested_ahead(P, Q):
    for factor, w_bf16, addend, out_bf16 in itertools.product((0, 1), repeat=4):
        assert b.fp4_gemm_tiling(P, Q, 0, factor, w_bf16, addend, out_bf16) == (64, 0, 0)


# (P, Q, Kc, factor, w_bf16, addend, tile): either side of the lines, and shapes that were measured far from them
LINES = [
    # the smallest outputs: 32 x 32, up to two a CU, three without the factor (test_gemm_split_route.py)
    (64, 2048, 2048, 0, 0, 1, 32), (512, 512, 256, 1, 0, 0, 32), (512, 1536, 4096, 0, 0, 0, 32), (512, 1568, 4096, 0, 0, 0, 128),
    # rows of whole 128-byte lines: one round of 64 x 64 tiles, two, three
    (512, 2048, 1280, 0, 0, 0, 64), (512, 2048, 1536, 0, 0, 0, 128), (520, 2048, 256, 0, 0, 0, 64), (520, 2048, 512, 0, 0, 0, 128),
    (1032, 2048, 256, 0, 0, 0, 128), (512, 2048, 3072, 1, 1, 0, 64), (512, 2048, 3328, 1, 1, 0, 128), (520, 2048, 768, 1, 1, 1, 64),
    (520, 2048, 1024, 1, 1, 1, 128), (1032, 2048, 256, 1, 0, 1, 64), (1032, 2048, 512, 1, 0, 1, 128),
    # others
    (192, 4128, 1216, 0, 0, 0, 64), (32, 704, 1056, 0, 0, 0, 64), (224, 3520, 1312, 0, 0, 1, 64), (64, 16384, 6144 - 32, 0, 0, 0, 64),
    (64, 16384, 6176, 0, 0, 0, 128), (520, 2048, 1056, 0, 0, 0, 64), (520, 2048, 1120, 0, 0, 0, 128),
    (1032, 2048, 416, 0, 0, 0, 64), (1032, 2048, 480, 0, 0, 0, 128), (1024, 832, 6016, 1, 1, 0, 64), (64, 16384, 8416, 1, 1, 0, 64),
    (64, 16384, 8480, 1, 1, 0, 128), (520, 2048, 1312, 1, 1, 0, 64), (1280, 1280, 2400, 1, 1, 0, 128), (1032, 2048, 1184, 1, 1, 0, 64), (1032, 2048, 1248, 1, 1, 0, 128),
    (1032, 2048, 1376, 1, 0, 0, 64), (672, 5496, 384, 1, 0, 0, 64), (672, 5496, 672, 1, 0, 0, 128),
    # what an XCD's tiles need of the operands beyond its L2
    (320, 3200, 2592, 0, 0, 0, 64), (320, 3200, 3616, 0, 0, 0, 128), (512, 2048, 3104, 0, 0, 0, 64), (512, 2048, 4640, 0, 0, 0, 128),
    (512, 4096, 1312, 1, 1, 1, 128), (512, 4096, 1184, 1, 1, 1, 64),
    # fp32 weights: two rounds of 128 x 128 tiles, three with an addend
    (2872, 3376, 8448, 1, 0, 0, 256), (2872, 3376, 8448, 1, 0, 1, 128), (1024, 8160, 8448, 1, 0, 0, 128),
]


@pytest.mark.parametrize("P,Q,Kc,factor,w_bf16,addend,tile", LINES)
def test_tiles(P, Q, Kc, factor, w_bf16, addend, tile):
    assert b.fp4_gemm_tiling(P, Q, Kc, factor, w_bf16, addend, 0, 256)[0] == tile


# (P, Q, Kc, factor, w_bf16, addend, out_bf16, whether the workgroups begin in quarters)
STAGGER = [
    (8192, 4864, 2048, 0, 0, 1, 1, True), (8192, 4864, 2048, 0, 0, 0, 1, False), (8192, 4864, 2048, 0, 0, 0, 0, True),   # 2.4 rounds
    (16384, 4096, 1024, 0, 0, 0, 0, False), (16384, 6144, 2048, 0, 0, 1, 0, False), (16384, 4096, 1024, 0, 0, 1, 1, True),   # whole rounds
    (16384, 4352, 1024, 0, 0, 0, 0, True),                                                                              # and cut tiles behind
    (8192, 5888, 256, 0, 0, 1, 1, False), (8192, 5888, 2048, 0, 0, 1, 1, True), (8192, 6144, 2048, 0, 0, 1, 1, False),   # nearly three rounds, three
    (8192, 5888, 4096, 1, 0, 1, 0, False), (16384, 4352, 256, 1, 1, 0, 0, False), (16384, 4352, 2048, 1, 1, 0, 0, True),     # the factor
    (8192, 2048, 4096, 0, 0, 1, 1, False),                                                                               # 128 x 128 tiles
]


@pytest.mark.parametrize("P,Q,Kc,factor,w_bf16,addend,out_bf16,on", STAGGER)
def test_late_workgroups(P, Q, Kc, factor, w_bf16, addend, out_bf16, on):
    assert (b.fp4_gemm_tiling(P, Q, Kc, factor, w_bf16, addend, out_bf16)[2] > 0) == on
