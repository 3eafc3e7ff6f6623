"""The levels of pending modification: launched together or one by one, by the number of rows and their length (k_pend_norm).  Whichever it is, a workgroup that looks in vain for the entries it builds on makes them itself, with the same bits."""
import numpy as np
import pytest

from parity_util import run_gpu, to_torch
from specgbv_synth import Workload, make_inputs
from test_gpu_pending import _state_tensor, check_pending

pytestmark = pytest.mark.gpu

# B, K, L, V, dtype, levels: launched together up to six row pairs per compute unit, and of given levels up to 6000 vectors a row
TOGETHER = [(3, 2, 5, 2049 * 4, "f32", 3), (5, 3, 4, 1029, "bf16", 2), (2, 2, 6, 4104, "bf16", 16),
            (4, 2, 4, 8 * 1023, "bf16", 2), (4, 2, 4, 8 * 1024, "bf16", 2)]       # (four parts a row, eight)
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
    for polls in ("0", "1"):                        # (all entries made alone; those that are not there yet)
        monkeypatch.setenv("SPECGBV_EXCESS_POLLS", polls)
        _same(waited, run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count)))


@pytest.mark.parametrize("B,K,L,V,dtype,full,together", [(4, 3, 6, 4104, "f32", False, True), (65, 4, 7, 520, "f32", False, False),
                                                          (65, 4, 7, 520, "f32", True, False), (130, 3, 5, 1030, "bf16", True, False),
                                                          (40, 4, 7, 1032, "bf16", True, True)])
def test_levels_of_a_state(B, K, L, V, dtype, full, together, monkeypatch):
    """As given levels; full: every level modifies every row.  together: there are as few row pairs as are launched together."""
    import torch
    import paper_2604_25925_amd as sg
    assert (B * K * L <= 6 * _compute_units()) == together
    t, d, tok, carry, count = _case(B, K, L, V, dtype, L - 1)
    if full:
        count[:] = L
    given = run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count))
    for polls in (None, "0", "1"):
        if polls is not None:
            monkeypatch.setenv("SPECGBV_EXCESS_POLLS", polls)
        state = _state_tensor(carry, count, B)
        acc, f, out, ws = sg.specgbv_verify_ex(to_torch(t), to_torch(d), to_torch(tok), 0.8, 4, 1, pending_state=state)
        torch.cuda.synchronize()
        got = dict(accepted_len=acc.cpu().numpy(), accepted_draft_idx=f.cpu().numpy(), out_tokens=out.cpu().numpy())
        got.update(sg.specgbv_read_intermediates(ws, B, K, L, V, 1 if dtype == "bf16" else 0))
        _same(got, given)


def _compute_units():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("V,dtype", [(1032, "bf16"), (520, "f32")])
@pytest.mark.parametrize("over", [0, 1])
def test_as_many_rows_as_are_launched_together(V, dtype, over, monkeypatch):
    """Five levels that modify every row of as many row pairs as their levels are launched together for, six per compute unit (twice
    what is resident at once), and of a prefix more, launched by level: given and as a state, and, of some prefixes, against the oracle."""
    import torch
    import paper_2604_25925_amd as sg
    K, L, levels = 4, 6, 5
    B = 6 * _compute_units() // (K * L) + over
    t, d, tok, _, _ = _case(B, K, L, V, dtype, levels)
    carry = np.random.default_rng(V).normal(2.0, 0.8, (levels, B))
    count = np.full((levels, B), L, np.int32)
    check_pending(t, d, tok, 0.8, 4, 1, carry, count, "all rows under five levels %s" % ((B, V, dtype),), gpu_slice=list(range(0, B, 11)))
    given = run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count))
    for polls in (None, "0", "1"):
        if polls is not None:
            monkeypatch.setenv("SPECGBV_EXCESS_POLLS", polls)
        acc, f, out, ws = sg.specgbv_verify_ex(to_torch(t), to_torch(d), to_torch(tok), 0.8, 4, 1, pending_state=_state_tensor(carry, count, B))
        torch.cuda.synchronize()
        got = dict(accepted_len=acc.cpu().numpy(), accepted_draft_idx=f.cpu().numpy(), out_tokens=out.cpu().numpy())
        got.update(sg.specgbv_read_intermediates(ws, B, K, L, V, 1 if dtype == "bf16" else 0))
        _same(got, given)


def test_empty_levels_take_no_parts():
    """One level of a state of eight, seven of them empty: its rows are shared among as many workgroups as those of the level alone
    (sixteen, of 1088 vectors each), which the bits of its normalisers show."""
    import torch
    import paper_2604_25925_amd as sg
    B, K, L, V = 1, 2, 9, 8 * 16 * 1088
    t, d, tok, carry, count = _case(B, K, L, V, "bf16", 1)
    count[:] = 4
    alone = run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count))
    ws = sg.specgbv_verify_ex(to_torch(t), to_torch(d), to_torch(tok), 0.8, 4, 1, pending_state=_state_tensor(carry, count, B))[3]
    torch.cuda.synchronize()
    got = sg.specgbv_read_intermediates(ws, B, K, L, V, 1)
    for key in ("lse_q", "log_nu", "s", "h"):
        assert np.array_equal(got[key], alone[key], equal_nan=True), key


@pytest.mark.parametrize("B,K,L,levels", [(1, 8, 2, 16), (1, 16, 1, 16), (2, 1, 2, 16), (1, 4, 17, 16)])
def test_room_for_the_parts_sums(B, K, L, levels, monkeypatch):
    """As many parts as fit: all levels' units of the first two have no room for eight parts a row, those of the others have."""
    t, d, tok, carry, count = _case(B, K, L, 8200, "bf16", levels)
    count[:] = L
    check_pending(t, d, tok, 0.8, 4, 1, carry[:2] + 1.5, count[:2], "room %s" % ((B, K, L),))
    waited = run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count))
    for polls in ("0", "1"):
        monkeypatch.setenv("SPECGBV_EXCESS_POLLS", polls)
        _same(waited, run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count)))


def _all_rows_under_all_levels(B, K, L, V, polls, calls=3):
    """Milliseconds of a call (the fastest of a few) whose state's L - 1 levels modify every row."""
    import os
    import torch
    import paper_2604_25925_amd as sg
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    t = torch.empty((B, K, L + 1, V), dtype=torch.bfloat16, device="cuda").normal_(0.0, 3.0, generator=gen)
    d = torch.empty((B, K, L, V), dtype=torch.bfloat16, device="cuda").normal_(0.0, 3.0, generator=gen)
    tok = torch.randint(V, (B, K, L), dtype=torch.int32, device="cuda", generator=gen)
    start = _state_tensor(np.full((L - 1, B), 0.5), np.full((L - 1, B), L, np.int32), B)
    best = []
    for p in polls:
        if p is None:
            os.environ.pop("SPECGBV_EXCESS_POLLS", None)
        else:
            os.environ["SPECGBV_EXCESS_POLLS"] = p
        times = []
        for _ in range(calls + 1):
            state = start.clone()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            sg.specgbv_verify_ex(t, d, tok, 0.8, 4, 1, pending_state=state)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        best.append(min(times[1:]))
    os.environ.pop("SPECGBV_EXCESS_POLLS", None)
    return best


# (a unit waits for fifteen levels, two milliseconds and more; for six, of the largest vocabularies)
@pytest.mark.parametrize("B,K,L,V", [(1, 4, 17, 1000000), (8, 8, 8, 256000)])
def test_long_rows_are_waited_for(B, K, L, V):
    """The looks outlast the levels below: no longer than with a thousand times as many (130 and 2.7 times as long where they did not)."""
    usual, many = _all_rows_under_all_levels(B, K, L, V, (None, "1048576"))
    assert usual < 1.5 * many


def test_entries_made_alone_cost_little():
    """With next to no looks a workgroup makes only what is still not there: twice the time (all of it again: 75 times)."""
    usual, few = _all_rows_under_all_levels(1, 4, 17, 128256, (None, "1"))
    assert few < 8 * usual


@pytest.mark.parametrize("polls", [None, "1"])
def test_ratios_that_are_no_numbers(polls, monkeypatch):
    """A carried NaN with all bits set, which is what an entry that is not there yet holds, as any other NaN."""
    if polls:
        monkeypatch.setenv("SPECGBV_EXCESS_POLLS", polls)
    t, d, tok, carry, count = _case(3, 2, 5, 2049 * 4, "f32", 3)
    count[:, 1] = 5
    carry[0, 1] = np.nan
    plain = run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count))
    carry[0, 1] = np.array([~np.uint64(0)]).view(np.float64)[0]
    _same(plain, run_gpu(t, d, tok, 0.8, 4, 1, pending=(carry, count)))
