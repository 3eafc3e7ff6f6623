"""The log-normalisers' logarithm, on rows whose sums are exact in float32 and need more than its 24 bits (needs an MI355X: run
with -m gpu)."""
import numpy as np
import pytest

from parity_util import to_torch

pytestmark = pytest.mark.gpu

T = 1.442695            # log2(e) / T is 1 in float32: a logit of -k weighs 2^-k


@pytest.mark.parametrize("dtype,V", [("f32", 1000), ("f32", 8192), ("f32", 30000), ("bf16", 8200), ("bf16", 32768)])
def test_kseq_rows_on_chip(dtype, V):
    """Logits 0 .. -14 or masked.  Sums below 2^15: half a unit in the last place of their log2 (8.9e-16) and the logarithm's own error
    (7e-16) times ln 2, and half a unit of the product (8.9e-16): 2.0e-15."""
    import torch
    import paper_2604_25925_amd as sg
    B, K, L = 32, 8, 2
    r = np.random.RandomState(V)
    rows = []
    for n_rows in (L + 1, L):
        z = -np.floor(r.uniform(0.0, 15.0, (B, K, n_rows, V)) ** 2 / 15.0).astype(np.float32)
        n = np.exp(r.uniform(0.0, np.log(V), (B, K, n_rows, 1)))
        z[np.arange(V) > n] = -np.inf
        rows.append(z)
    want = [np.log(np.exp2(z[:, :, :L].astype(np.float64)).sum(axis=3)) for z in rows]
    if dtype == "bf16":
        rows = [(z.view(np.uint32) >> 16).astype(np.uint16) for z in rows]
    tl, dl = (to_torch(z) for z in rows)
    ws = sg.specgbv_verify_kseq(tl, dl, torch.zeros((B, K, L), dtype=torch.int32, device="cuda"), T, 1, 0)[-1]
    torch.cuda.synchronize()
    got = sg.specgbv_read_intermediates(ws, B, K, L, V, 1 if dtype == "bf16" else 0)
    for ln, key in zip(want, ("lse_q", "lse_p")):
        err = np.abs(np.asarray(got[key]).reshape(B, K, L) - ln)
        print(key, "largest error %.2e" % err.max())
        assert err.max() <= 2.0e-15, key
