"""The final token of rows of more than 163840 entries, whose partial sums a whole workgroup adds up before one wave searches
them, at the sizes where that begins and where a thread's share changes (needs an MI355X: run with -m gpu)."""
import numpy as np
import pytest

from parity_util import check_case
from specgbv_synth import Workload, f32_to_bf16_bits, make_inputs
from test_gpu_comparison import check
from test_gpu_pending import check_pending

pytestmark = pytest.mark.gpu


def _inputs(B, K, L, V, dtype):
    return make_inputs(Workload("long", B, K, L, V, dtype, 2.5, 0.9, head=50, temperature=0.8), seed=V % 1000)


@pytest.mark.parametrize("B,K,L,V,dtype", [
    (3, 1, 2, 163840, "bf16"), (3, 1, 2, 163841, "bf16"),          # 320 segments of 512, and 321: 2 per thread
    (2, 1, 2, 262144, "f32"), (2, 1, 2, 262145, "bf16"),           # 2 per thread, and 3
    (2, 1, 2, 524288, "bf16"), (2, 1, 2, 524801, "bf16"),          # a thread's first load of four, and one more
    (1, 1, 2, 1000003, "f32"), (1, 2, 1, 3000001, "bf16"),         # a lane's chunk of 64 segments, and of more
])
def test_long_rows(B, K, L, V, dtype):
    t, d, tok = _inputs(B, K, L, V, dtype)
    for offset in range(4):                                        # other uniforms: other segments
        check_case(t, d, tok, 0.8, 3, offset, "auto", "long rows %s" % ((B, K, L, V, dtype),))


def test_mass_in_one_segment_and_equal_rows():
    """Most segments masked, so that few of a thread's have any weight; and a draft equal to the target, whose residual
    vanishes everywhere (the token is drawn from the target row)."""
    t, d, tok = _inputs(3, 1, 1, 400001, "f32")
    t[0, :, :, :390000] = -np.inf
    d[0, :, :, :390000] = -np.inf
    t[1, :, :, 3000:] = -np.inf
    d[1, :, :, 3000:] = -np.inf
    d[2, 0, 0] = t[2, 0, 0]
    tok[0], tok[1] = 395000, 17
    for offset in range(4):
        check_case(t, d, tok, 0.8, 3, offset, "auto", "long masked rows")
    check_case(f32_to_bf16_bits(t), f32_to_bf16_bits(d), tok, 0.8, 3, 9, "auto", "long masked rows bf16")


def test_other_entry_points():
    t, d, tok = _inputs(2, 2, 3, 200003, "bf16")
    check(t, d, tok, 0.8, 3, 1, None, "K-SEQ long rows", rho_tol=3.0)
    check_pending(t, d, tok, 0.8, 3, 1, np.array([0.3, -0.2]), np.array([2, 1], np.int32), "pending long rows")
