"""Which residual products are gathered (csrc/spmm_gather.hip), on the CPU: by how many entries there can be, not by the sizes alone."""
import itertools

import pytest

from paper_2501_17116_amd import binding as b

BF16, F32 = b.FP4_BF16, b.FP4_F32

# shapes at which both sides were measured: the share of entries up to which the gather was faster, and one from which it was slower
LINES = [
    (BF16, 4096, 512, 1024, 0.12, 0.20), (BF16, 2048, 1024, 1024, 0.12, 0.20), (BF16, 1056, 1376, 2080, 0.09, 0.20),
    (BF16, 2048, 2048, 1024, 0.09, 0.20), (BF16, 2048, 2048, 2048, 0.06, 0.09), (BF16, 1024, 4096, 1024, 0.12, 0.50),
    (BF16, 512, 8192, 1024, 0.12, 0.50), (BF16, 1024, 1024, 1024, 0.20, 0.50), (F32, 4096, 512, 1024, 0.20, 0.50),
    (F32, 2048, 2048, 2048, 0.12, 0.20),
]


@pytest.mark.parametrize("dt,P,Q,N,faster,slower", LINES)
def test_dense_matrices_are_not_gathered(dt, P, Q, N, faster, slower):
    assert b.fp4_residual_spmm_gathers(P, Q, N, dt, int(faster * P * Q))
    assert not b.fp4_residual_spmm_gathers(P, Q, N, dt, int(slower * P * Q))
    assert not b.fp4_residual_spmm_gathers(P, Q, N, dt, 2 ** 63 - 1)      # a full one, for all that is known


@pytest.mark.parametrize("dt,P,Q,N", [(F32, 1024, 1024, 1024), (F32, 1056, 1376, 2080), (F32, 512, 4096, 1024), (BF16, 64, 2048, 2048),
                                      (BF16, 512, 512, 512), (F32, 256, 512, 512)])
def test_where_even_a_full_one_is(dt, P, Q, N):
    assert b.fp4_residual_spmm_gathers(P, Q, N, dt, P * Q)


def test_never_for_more_entries_only():
    for dt, P, Q, N in itertools.product((BF16, F32), (32, 1056, 4096, 16384), (32, 1376, 8192, 8224), (8, 1024, 8192)):
        took = [b.fp4_residual_spmm_gathers(P, Q, N, dt, int(s * P * Q)) for s in (0.0, 0.002, 0.02, 0.06, 0.12, 0.2, 0.5, 1.0)]
        assert took == sorted(took, reverse=True)
        if P * Q * N > 2 ** 33 or Q > 8192:
            assert not any(took)
