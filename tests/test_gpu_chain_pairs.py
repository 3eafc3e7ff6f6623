"""The chain schedule with two workgroups per compute unit, at the sizes where that ends (needs an MI355X: run with
-m gpu)."""
import pytest

from parity_util import check_case
from specgbv_synth import Workload, make_inputs

pytestmark = pytest.mark.gpu


def _inputs(B, K, L, V, dtype, T=0.8, seed=5, sigma=2.5):
    return make_inputs(Workload("rows", B, K, L, V, dtype, sigma, 0.9, head=min(20, V // 4), temperature=T), seed=seed)


@pytest.mark.parametrize("B,K,L,V,dtype", [
    (30, 9, 2, 28672, "bf16"),       # 270 chains: 14 compute units hold two; seven slots, none in LDS
    (66, 8, 2, 14340, "f32"),        # 528 chains on 512 workgroups: two chains for the first sixteen; ragged eighth slot
    (33, 8, 2, 45056, "bf16"),       # rows of exactly 7 + 4 slots
    (33, 8, 2, 45064, "bf16"),       # one vector more: a workgroup per compute unit
])
def test_two_chains_per_compute_unit(B, K, L, V, dtype):
    t, d, tok = _inputs(B, K, L, V, dtype)
    check_case(t, d, tok, 0.8, 3, 1, "chain", "shared unit %s" % ((B, K, L, V, dtype),))
