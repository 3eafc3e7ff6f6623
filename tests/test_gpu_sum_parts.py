"""Sums of Eq. (hik) of rows in parts, with and without pending levels: parts of less than one vector per thread (the first loads
of the lanes beyond them are repeats of the last vector), of one and two per thread and one vector more, whole and ragged
(needs an MI355X: run with -m gpu)."""
import numpy as np
import pytest

from parity_util import check_case
from specgbv_synth import Workload, make_inputs
from test_gpu_pending import check_pending

pytestmark = pytest.mark.gpu

# two rows with a sum, so 16 parts each: of 128, 129, 512, 513 and 1024 vectors, and one vector in the last step of a sweep
SIZES = [("f32", 8192), ("f32", 8195), ("f32", 32768), ("f32", 32772), ("f32", 65536), ("f32", 65603), ("bf16", 8200), ("bf16", 65536),
         ("bf16", 65549), ("bf16", 131080)]


@pytest.mark.parametrize("dtype,V", SIZES)
@pytest.mark.parametrize("levels", [0, 1, 2])
def test_parts(dtype, V, levels):
    t, d, tok = make_inputs(Workload("parts", 1, 2, 2, V, dtype, 2.0, 0.8, head=8, temperature=0.9), seed=V % 83)
    tok[0, 1, 1] = V - 1
    if levels == 0:
        check_case(t, d, tok, 0.9, 3, 1, "split", "sums in parts %d %s" % (V, dtype))
    else:
        carry, count = np.array([[0.2], [-0.3]])[:levels], np.array([[1], [2]], np.int32)[-levels:]
        check_pending(t, d, tok, 0.9, 3, 1, carry, count, "sums in parts under %d levels %d %s" % (levels, V, dtype))
