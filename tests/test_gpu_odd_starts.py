"""Vectors of bfloat16 rows that start at an odd entry are loaded from the entry in front on and put together (two-pass schedule): the rows' first and
last entries decide (drafted tokens there, and entries in front that would change every sum), with and without parts, and
with tensors that themselves start at an odd entry.  Where a row starts makes no difference to a bit of its results."""
import numpy as np
import pytest

from parity_util import check_case, to_torch
from specgbv_synth import Workload, f32_to_bf16_bits, make_inputs
from test_gpu_pending import check_pending

pytestmark = pytest.mark.gpu


def _inputs(B, K, L, V):
    """Every row's last entry, which lies in front of the next row, holds a good part of its mass, and drafted tokens are
    first and last entries."""
    t, d, tok = make_inputs(Workload("starts", B, K, L, V, "f32", 2.0, 0.8, head=8, temperature=0.9), seed=V)
    t[..., V - 1], d[..., V - 1] = t.max() + 1.0, d.max() + 1.0
    tok[:, 0, ::2], tok[:, -1, 1::2] = 0, V - 1
    return f32_to_bf16_bits(t), f32_to_bf16_bits(d), tok


# (4097 .. 4103: every remainder of an odd row, one vector per thread and a little; 8199 with few rows: parts)
@pytest.mark.parametrize("B,K,L,V", [(3, 3, 4, V) for V in (4097, 4099, 4101, 4103)] + [(1, 2, 4, 8199), (1, 3, 3, 32771), (64, 3, 6, 8193)])
def test_two_pass(B, K, L, V):
    t, d, tok = _inputs(B, K, L, V)
    check_case(t, d, tok, 0.9, 4, 1, "split", "odd starts %s" % ((B, K, L, V),))


@pytest.mark.parametrize("B,K,L,V", [(3, 3, 4, 4101), (2, 2, 4, 8199)])
def test_under_levels(B, K, L, V):
    t, d, tok = _inputs(B, K, L, V)
    rng = np.random.default_rng(V)
    check_pending(t, d, tok, 0.9, 4, 1, rng.normal(0, 0.5, (2, B)), rng.integers(0, L + 1, (2, B)).astype(np.int32), "odd starts %d" % V)


def _run(tl, dl, tok, **how):
    import torch
    import paper_2604_25925_amd as sg
    B, K, L, V = dl.shape
    out = sg.specgbv_verify_ex(tl, dl, to_torch(tok), 0.9, 4, 1, algo="split", **how)
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out[:3]], sg.specgbv_read_intermediates(out[3], B, K, L, V, 1)


# (an even vocabulary, whose rows all start as the tensor does: with whole vectors, without, and in parts)
@pytest.mark.parametrize("B,K,L,V", [(3, 3, 4, 4103), (1, 2, 4, 8199), (3, 3, 4, 4104), (3, 3, 4, 4098), (1, 2, 4, 8200), (1, 2, 4, 8194)])
@pytest.mark.parametrize("levels", [0, 2])
def test_tensors_that_start_at_an_odd_entry(B, K, L, V, levels):
    """The parity of every row is the other one."""
    import torch

    def run(shift):
        def moved(x):
            flat = torch.full((x.numel() + 1,), 100.0, dtype=x.dtype, device=x.device)      # (what lies in front of the tensor)
            flat[shift:shift + x.numel()] = x.reshape(-1)
            return flat[shift:shift + x.numel()].view(x.shape)
        return _run(moved(tl), moved(dl), tok, pending=pend)

    t, d, tok = _inputs(B, K, L, V)
    tl, dl = to_torch(t), to_torch(d)
    rng = np.random.default_rng(V)
    pend = (torch.from_numpy(rng.normal(0, 0.5, (levels, B))).cuda(),
            torch.from_numpy(rng.integers(0, L + 1, (levels, B)).astype(np.int32)).cuda()) if levels else None
    (o0, i0), (o1, i1) = run(0), run(1)
    for a, b in zip(o0, o1):
        assert np.array_equal(a, b)
    for key in i0:
        assert np.array_equal(i0[key], i1[key], equal_nan=True), key


@pytest.mark.parametrize("B,K,L,V", [(2, 4, 3, 4101), (1, 3, 4, 8199), (20, 8, 3, 8193)])
def test_equal_rows(B, K, L, V):
    """Drafts that are copies of one another, whose rows start at even and odd entries in turn."""
    t, d, tok = _inputs(B, K, L, V)
    t, d, tok = (np.ascontiguousarray(np.repeat(x[:, :1], K, axis=1)) for x in (t, d, tok))
    _, res = _run(to_torch(t), to_torch(d), tok)
    for key in ("lse_q", "lse_p", "log_nu", "s"):
        assert np.array_equal(res[key], np.repeat(res[key][:, :1], K, axis=1), equal_nan=True), key
