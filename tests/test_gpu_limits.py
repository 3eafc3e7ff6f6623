"""The largest accepted number of table entries per prefix, K L = 1024 (and K L = 992 with the most rows): the decision takes
several visits per thread and 75 KB of LDS there (needs an MI355X: run with -m gpu)."""
import numpy as np
import pytest

import test_gpu_peaked_rows as peaked
from parity_util import check_case
from specgbv_synth import Workload, make_inputs
from test_gpu_comparison import check
from test_gpu_pending import check_pending

pytestmark = pytest.mark.gpu

SHAPES = [(2, 64, 16, 64), (2, 16, 62, 40), (1, 64, 16, 2049)]


def _inputs(B, K, L, V):
    return make_inputs(Workload("limit", B, K, L, V, "f32", 2.0, 0.8, head=8, temperature=1.0), seed=2)


@pytest.mark.parametrize("B,K,L,V", SHAPES)
@pytest.mark.parametrize("algo", ["auto", "split"])
def test_verify(B, K, L, V, algo):
    t, d, tok = _inputs(B, K, L, V)
    check_case(t, d, tok, 1.0, 3, 1, algo, "limits %s" % ((B, K, L, V),))


@pytest.mark.parametrize("B,K,L,V", SHAPES)
def test_kseq(B, K, L, V):
    t, d, tok = _inputs(B, K, L, V)
    check(t, d, tok, 1.0, 3, 1, None, "K-SEQ limits %s" % ((B, K, L, V),), rho_tol=3.0)


@pytest.mark.parametrize("B,K,L,V", SHAPES[:2])
def test_pending(B, K, L, V):
    t, d, tok = _inputs(B, K, L, V)
    check_pending(t, d, tok, 1.0, 3, 1, np.linspace(-0.3, 0.4, B), np.array([L - 1, 3], np.int32), "pending limits %s" % ((B, K, L, V),))


@pytest.mark.parametrize("algo,V", [("split", 300), ("auto", 2049), ("auto", 300)])
def test_rows_that_need_the_cancellation_free_sum(algo, V):
    """Hundreds of marked rows of one prefix, more than fit one round of the final-token kernel's wait."""
    peaked.test_block_ratio_runs_away(algo, "f32", V, 3, 64, 16)
