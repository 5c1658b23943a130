"""The kernels of large residual products (csrc/spmm_mfma.hip, csrc/spmm.hip) at small sizes, which fp4_residual_spmm itself gives to
the gathering kernel: every check of the residual product once more through fp4_residual_spmm_general."""
import pytest

from paper_2501_17116_amd import binding as b
from test_gpu_parity import (test_residual_spmm, test_residual_spmm_many_long_rows, test_residual_spmm_random_shapes,  # noqa: F401
                             test_residual_spmm_with_long_rows)
from test_gpu_spmm_mfma import *  # noqa: F401,F403
from test_gpu_spmm_rows import test_against_fp64 as test_fp32_against_fp64, test_no_columns  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _general(monkeypatch):
    monkeypatch.setattr(b, "fp4_residual_spmm", b.fp4_residual_spmm_general)
