"""K-SEQ rows kept in registers, at the edges of their two tiles (16 and 64 entries for each of 512 threads) and with
every remainder of a vector, against the oracle (needs an MI355X: run with -m gpu)."""
import pytest

from specgbv_synth import Workload, make_inputs
from test_gpu_comparison import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K,L,V,dtype", [
    (3, 4, 2, 8, "bf16"), (3, 4, 2, 13, "bf16"), (3, 4, 2, 4, "f32"), (3, 4, 2, 7, "f32"), (3, 4, 2, 3, "f32"),
    (2, 4, 3, 8192, "bf16"), (2, 4, 3, 8193, "bf16"), (2, 4, 3, 8191, "f32"), (2, 4, 3, 8195, "f32"),
    (2, 4, 3, 32768, "bf16"), (2, 4, 3, 32761, "bf16"), (2, 4, 3, 32769, "bf16"), (2, 4, 3, 32766, "f32"), (2, 4, 3, 32772, "f32"),
])
def test_tiles(B, K, L, V, dtype):
    t, d, tok = make_inputs(Workload("kseq", B, K, L, V, dtype, 2.5, 0.8, head=min(8, V // 2), temperature=0.8), seed=3)
    check(t, d, tok, 0.8, 3, 1, None, "K-SEQ tiles %s" % ((B, K, L, V, dtype),), rho_tol=3.0)


@pytest.mark.parametrize("B,L,V,sigma_d,T,seed", [(64, 4, 301, 1.0, 0.4, 5), (64, 3, 100, 0.25, 0.3, 1)])
def test_roots_behind_a_change_of_slope(B, L, V, sigma_d, T, seed):
    """Low temperatures: one entry holds nearly all mass, and the equation for rho turns flat by orders of magnitude as
    rho p passes q there, so that a short Newton step in front of that point says nothing about the root."""
    t, d, tok = make_inputs(Workload("kink", B, 4, L, V, "bf16", 3.0, sigma_d, head=min(50, V // 4), temperature=T), seed=seed)
    check(t, d, tok, T, 1, 1, None, "K-SEQ roots behind a change of slope V=%d" % V)
