"""The levels of pending modification: launched together or one by one, by the number of rows and their length (k_pend_norm).  Whichever it is, a workgroup that looks in vain for the entries it builds on makes them itself, with the same bits."""
import numpy as np
import pytest

from parity_util import run_gpu, to_torch
from specgbv_synth import Workload, make_inputs
from test_gpu_pending import _state_tensor, check_pending

pytestmark = pytest.mark.gpu

# B, K, L, V, dtype, levels
TOGETHER = [(3, 2, 5, 2049 * 4, "f32", 3), (5, 3, 4, 1029, "bf16", 2), (2, 2, 6, 4104, "bf16", 16)]
BY_LEVEL = [(65, 4, 6, 1032, "bf16", 3), (2, 1, 3, 48008, "bf16", 2)]


def _case(B, K, L, V, dtype, levels):
    t, d, tok = make_inputs(Workload("levels", B, K, L, V, dtype, 2.5, 0.8, head=20, temperature=0.8), seed=17)
    rng = np.random.default_rng(levels)
    return t, d, tok, rng.normal(0.5, 0.8, (levels, B)), rng.integers(0, L + 1, (levels, B)).astype(np.int32)


def _same(a, b):
    assert a.keys() == b.keys()
    for key in a:
        assert np.array_equal(a[key], b[key], equal_nan=True), key


@pytest.mark.parametrize("B,K,L,V,dtype,levels", TOGETHER + BY_LEVEL)
def test_given_levels(B, K, L, V, dtype, levels, monkeypatch):
    t, d, tok, carry, count = _case(B, K, L, V, dtype, levels)
    if levels < 4:                                  # (a few prefixes: check_pending allows one that the oracle cannot decide either)
        check_pending(t, d, tok, 0.8, 4, 1, carry, count, "levels %s" % ((B, K, L, V, dtype, levels),), gpu_slice=list(range(min(B, 8))))
    waited = run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count))
    monkeypatch.setenv("SPECGBV_EXCESS_POLLS", "0")
    _same(waited, run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count)))


@pytest.mark.parametrize("B,K,L,V,dtype,full", [(4, 3, 6, 4104, "f32", False), (65, 4, 7, 520, "f32", False), (65, 4, 7, 520, "f32", True),
                                                 (130, 3, 5, 1030, "bf16", True)])
def test_levels_of_a_state(B, K, L, V, dtype, full, monkeypatch):
    """As given levels; full: every level modifies every row."""
    import torch
    import paper_2604_25925_amd as sg
    t, d, tok, carry, count = _case(B, K, L, V, dtype, L - 1)
    if full:
        count[:] = L
    given = run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count))
    for polls in (None, "0"):
        if polls is not None:
            monkeypatch.setenv("SPECGBV_EXCESS_POLLS", polls)
        state = _state_tensor(carry, count, B)
        acc, f, out, ws = sg.specgbv_verify_ex(to_torch(t), to_torch(d), to_torch(tok), 0.8, 4, 1, pending_state=state)
        torch.cuda.synchronize()
        got = dict(accepted_len=acc.cpu().numpy(), accepted_draft_idx=f.cpu().numpy(), out_tokens=out.cpu().numpy())
        got.update(sg.specgbv_read_intermediates(ws, B, K, L, V, 1 if dtype == "bf16" else 0))
        _same(got, given)
