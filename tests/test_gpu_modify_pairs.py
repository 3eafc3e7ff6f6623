"""Modified row pairs of Algorithm 2, whose workgroups keep 6 or 9 vector pairs per thread and read the rest of the pair again:
both sides of those edges, whole vectors and a repeated end, and rows whose weights all vanish (needs an MI355X: run with -m gpu)."""
import numpy as np
import pytest

from specgbv_synth import Workload, make_inputs
from test_gpu_modification import _check_modify

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,dtype", [
    (24576, "bf16"), (24577, "bf16"), (12288, "f32"), (12290, "f32"),      # 6 slots of 512 vectors, and one vector more
    (36864, "bf16"), (36872, "bf16"), (36869, "bf16"),                     # 9 slots; one vector read again, whole and ragged
    (18432, "f32"), (22528, "f32"), (22531, "f32"),                        # ...; two slots read again, and one vector of a third
])
def test_pairs(V, dtype):
    t, d, tok = make_inputs(Workload("pairs", 2, 2, 3, V, dtype, 2.0, 0.8, head=8, temperature=0.9), seed=V % 97)
    t = np.ascontiguousarray(t[:, :, :3])
    tok[:, 0, -1] = V - 1
    d[0, :, 0] = t[0, :, 0]                                # with a carried ratio of one: every weight of these rows is zero
    _, ora = _check_modify(t, d, tok, 0.9, np.array([0.0, -0.4]), np.array([2, 3], np.int32), "modified pairs %d %s" % (V, dtype))
    assert ora["fallback"][0, :, 0].all() and not ora["fallback"][:, :, 1:].all()


@pytest.mark.parametrize("V", [9216, 9224, 9216 + 256, 9216 + 264, 9216 + 504, 9216 + 512, 9216 + 768, 24576 + 8 * 31, 24576 + 8 * 33,
                               36864 + 8 * 40, 131072 + 8 * 63])
def test_half_vectors(V):
    """Whole bfloat16 rows of more than 9216 entries are dealt out in half vectors, 256 entries apart: last blocks of 512 entries
    without a second half, with a part of the first, with a part of the second, and whole, beside rows read for their
    log-probabilities alone."""
    t, d, tok = make_inputs(Workload("halves", 2, 2, 2, V, "bf16", 2.0, 0.8, head=8, temperature=0.9), seed=V % 89)
    t = np.ascontiguousarray(t[:, :, :2])
    tok[:, 0, -1] = V - 1
    _check_modify(t, d, tok, 0.9, np.array([-0.3, 0.2]), np.array([2, 1], np.int32), "half vectors %d" % V)
