"""Draft-side sampling at the edges of its segments and batches and at odd addresses, against the oracle (needs an
MI355X: run with -m gpu)."""
import numpy as np
import pytest

from specgbv_synth import f32_to_bf16_bits
from test_gpu_sampling import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,V", [
    (9, 1), (9, 7), (9, 8), (9, 9), (9, 511), (9, 512), (9, 513),
    (5, 65536), (5, 65537), (5, 32769),     # one batch of 8 waves, of 16 waves, and one entry more
    (3, 131072), (3, 131079), (2, 1048573), # 16 waves x 16 segments exactly, ragged, the longest rows
    (300, 4099),                            # more rows than compute units
])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_edges(rows, V, dtype):
    rng = np.random.default_rng(V)
    z = rng.normal(0, 2.5, (rows, V)).astype(np.float32)
    z[:, -1] += 3.0                                       # the row's last entry is drawn now and then
    if dtype == "bf16":
        z = f32_to_bf16_bits(z)
    _check(z, 0.8, 11, 2, 3, "sample edges %s" % ((rows, V, dtype),))
