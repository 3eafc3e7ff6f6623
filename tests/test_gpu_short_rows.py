"""Rows of up to 1024 entries in drafts of up to 8 rows, and of up to 2048 in up to 16 with many drafts, which one workgroup
per draft takes in one launch, at the sizes where that ends (needs an MI355X: run with -m gpu)."""
import pytest

import test_gpu_peaked_rows as peaked
from parity_util import check_case
from specgbv_synth import Workload, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K,L,V,dtype", [
    # one vector and less than two, one load per lane and two, the last size with few drafts and the first that is not in it
    (2, 2, 3, 8, "bf16"), (2, 2, 3, 9, "bf16"), (2, 2, 3, 4, "f32"), (1, 3, 2, 257, "f32"), (3, 2, 4, 512, "bf16"),
    (3, 2, 4, 519, "bf16"), (3, 4, 5, 1021, "f32"), (3, 2, 8, 1024, "bf16"), (3, 2, 4, 1025, "bf16"), (2, 2, 9, 1000, "f32"),
    # a draft of one row; many drafts: the longest, one row and one entry more
    (2, 1, 1, 1000, "bf16"), (65, 4, 16, 2048, "bf16"), (65, 4, 17, 2041, "bf16"), (130, 2, 9, 2047, "f32"), (130, 2, 9, 2049, "f32"),
    (600, 2, 3, 100, "bf16"),
])
def test_short_rows(B, K, L, V, dtype):
    t, d, tok = make_inputs(Workload("short", B, K, L, V, dtype, 2.5, 0.9, head=max(1, min(20, V // 4)), temperature=0.8), seed=5)
    tok[:, 0, -1] = V - 1                                  # a drafted token in the vector that is not whole
    check_case(t, d, tok, 0.8, 3, 1, "auto", "short rows %s" % ((B, K, L, V, dtype),))


@pytest.mark.parametrize("V,dtype,B,K,L", [(1001, "bf16", 4, 2, 5), (1002, "f32", 2, 3, 8), (2003, "f32", 130, 2, 8)])
def test_short_rows_that_need_the_cancellation_free_sum(V, dtype, B, K, L):
    peaked.test_block_ratio_runs_away("auto", dtype, V, B, K, L)
