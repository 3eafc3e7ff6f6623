"""The row-at-a-time schedule (the default where there are too few drafts for a workgroup each) at the sizes where its
tiles end (needs an MI355X: run with -m gpu).

The default takes the row schedule here: rows of at least one vector, too short or too few for the chain kernel, more
than half as many row pairs as compute units or rows of 512 vectors and more, and no more workgroups than two per compute
unit or, beyond that, parts that fill their tile.  Cases at the edges of what it takes, which go to its neighbours, say so.
"""
import numpy as np
import pytest

import test_gpu_peaked_rows as peaked
from parity_util import check_case
from specgbv_synth import Workload, make_inputs

pytestmark = pytest.mark.gpu


def _inputs(B, K, L, V, dtype, T=0.8, seed=5, sigma=2.5):
    return make_inputs(Workload("rows", B, K, L, V, dtype, sigma, 0.9, head=min(20, V // 4), temperature=T), seed=seed)


@pytest.mark.parametrize("B,K,L,V,dtype", [
    # (rows of one and two vectors, which k_short_rows takes)
    (11, 3, 4, 8, "bf16"), (11, 3, 4, 9, "bf16"), (11, 3, 4, 15, "bf16"), (17, 4, 2, 4, "f32"), (17, 4, 2, 7, "f32"),
    # the edges of the three tiles (1024, 2048 and 4096 vectors) and of the parts, with and without a remainder
    (5, 4, 8, 8192, "bf16"), (5, 4, 8, 8193, "bf16"), (5, 4, 8, 16384, "bf16"), (5, 4, 8, 16391, "bf16"),
    (9, 4, 8, 32767, "bf16"), (9, 4, 8, 32768, "bf16"), (9, 4, 8, 32769, "bf16"), (9, 4, 8, 16387, "f32"),
    # few rows: up to sixteen parts; parts that end in the middle of a slot; long rows in eight and sixteen parts (the last
    # case, one vector too long for them, goes to the two-pass kernels)
    (1, 1, 2, 4096, "bf16"), (1, 3, 3, 65543, "bf16"), (1, 2, 4, 300007, "bf16"), (2, 1, 2, 262145, "f32"),
    # a single row per draft (no Eq. (hik) sum at all; k_short_rows), and the longest drafts
    (140, 1, 1, 1003, "bf16"), (1, 3, 62, 2051, "f32"),
    # whole rows in the tiles of 1024, 1536, 2048 and 4096 vectors (288 row pairs: one part each)
    (9, 4, 8, 8192, "bf16"), (9, 4, 8, 8193, "bf16"), (9, 4, 8, 12288, "bf16"), (9, 4, 8, 12289, "bf16"),
    (9, 4, 8, 16384, "bf16"), (9, 4, 8, 16391, "bf16"), (9, 4, 8, 6143, "f32"), (9, 4, 8, 6145, "f32"),
    # rows of one and two vectors in drafts longer than k_short_rows takes (180 row pairs)
    (5, 4, 9, 8, "bf16"), (5, 4, 9, 16, "bf16"), (5, 4, 9, 4, "f32"), (5, 4, 9, 8, "f32"),
    # more workgroups than are resident, whose parts fill the tile; sixteen parts of 4096 vectors
    (9, 4, 8, 56009, "bf16"), (9, 4, 8, 23003, "f32"), (2, 1, 2, 262141, "f32"), (4, 4, 8, 32769, "bf16"),
    # a single row per draft, longer than k_short_rows takes
    (140, 1, 1, 1032, "bf16"), (140, 1, 1, 4099, "bf16"),
])
def test_rows_at_the_edges_of_tiles_and_parts(B, K, L, V, dtype):
    t, d, tok = _inputs(B, K, L, V, dtype)
    check_case(t, d, tok, 0.8, 3, 1, "auto", "rows %s" % ((B, K, L, V, dtype),))


@pytest.mark.parametrize("V,dtype", [(20003, "bf16"), (10002, "f32"), (70001, "bf16")])
def test_first_entries_masked_or_far_below_the_rest(V, dtype):
    """A lane's running reference starts without a finite entry, and is raised a hundred base-2 units and more on the way:
    the first third of a row is masked in one draft's rows and lies that far below the rest in the next one's."""
    t, d, tok = _inputs(4, 4, 5, V, "f32", T=0.3)
    n = V // 3
    tok = np.maximum(tok, n + 1).astype(np.int32) % V
    t[:, 1, :, :n], d[:, 1, :, :n] = -np.inf, -np.inf
    t[:, 2, :, :n] -= 40.0
    d[:, 2, :, :n] -= 35.0
    t[:, 3, :, ::2] = -np.inf
    tok[:, 3] |= 1
    t[:, :, :, V - 1], d[:, :, :, V - 1] = 1.0, 0.5
    tok = np.minimum(tok, V - 1)
    if dtype == "bf16":
        from specgbv_synth import f32_to_bf16_bits
        t, d = f32_to_bf16_bits(t), f32_to_bf16_bits(d)
    check_case(t, d, tok, 0.3, 9, 2, "auto", "masked rows V=%d %s" % (V, dtype))


@pytest.mark.parametrize("B,K,L,V,dtype", [(9, 4, 8, 9001, "bf16"), (1, 2, 6, 65543, "bf16")])
def test_bounded_wait_falls_back_to_the_waiting_workgroups_own_statistics(B, K, L, V, dtype, monkeypatch):
    """With no look at all at what the other workgroups leave, every workgroup computes the statistics of its draft's
    earlier rows (and of its row's other parts) itself; the results have the same bits."""
    from parity_util import run_gpu
    t, d, tok = _inputs(B, K, L, V, dtype)
    _, waited, _ = check_case(t, d, tok, 0.8, 3, 1, "auto", "rows, waiting")
    monkeypatch.setenv("SPECGBV_EXCESS_POLLS", "0")
    alone = run_gpu(t, d, tok, 0.8, 3, 1, "auto")
    for key in waited:
        assert np.array_equal(waited[key], alone[key], equal_nan=True), key


@pytest.mark.parametrize("V,dtype,B,K,L", [(9001, "bf16", 20, 2, 5), (16387, "f32", 12, 3, 4), (131077, "bf16", 2, 2, 4)])
def test_rows_that_need_the_cancellation_free_sum(V, dtype, B, K, L):
    peaked.test_block_ratio_runs_away("auto", dtype, V, B, K, L)


@pytest.mark.parametrize("V,T", [(8000, 0.7), (9001, 0.4), (16000, 0.7)])
def test_normalisers_are_as_accurate_as_on_the_two_pass_schedule(V, T):
    """Rms error of the ln-normalisers of 1024 rows against float64.  No more entries share a reference than on the two-pass
    schedule, so the errors have the same size; a tenth is left for the scatter of an rms over 1024 rows (3 %), and where the
    two-pass kernels add up other entries together."""
    import torch
    from parity_util import run_gpu, to_torch
    from specgbv_synth import f32_to_bf16_bits
    B, K, L = 32, 4, 4
    rng = np.random.default_rng(V)
    t = f32_to_bf16_bits(rng.normal(0, 3, (B, K, L + 1, V)).astype(np.float32))
    d = f32_to_bf16_bits(rng.normal(0, 3, (B, K, L, V)).astype(np.float32))
    tok = rng.integers(0, V, (B, K, L)).astype(np.int32)
    c = float(np.float32(1.4426950408889634 / float(np.float32(T)))) * 0.693147180559945309417
    ref = [torch.logsumexp(to_torch(np.ascontiguousarray(z)).double() * c, -1).cpu().numpy() for z in (t[:, :, :L], d)]
    rms = {}
    for algo in ("auto", "split"):
        g = run_gpu(t, d, tok, T, 1, 1, algo)
        rms[algo] = float(np.sqrt(np.mean([np.square(g["lse_q"] - ref[0]), np.square(g["lse_p"] - ref[1])])))
    print("[normalisers] V=%d T=%g: rms %r" % (V, T, rms), flush=True)
    assert rms["auto"] <= 1.1 * rms["split"]


def test_two_streams_at_once():
    """Calls of the rows schedule on two streams, each with its own workspace, beside calls that fill the GPU: whatever the
    order in which workgroups come to run, the results have the bits of the calls made alone."""
    import torch
    import paper_2604_25925_amd as sg
    from parity_util import to_torch
    shapes = [(9, 4, 8, 9001, "bf16"), (1, 3, 8, 65543, "bf16"), (8, 4, 5, 32000, "f32")]
    cases = []
    for i, shape in enumerate(shapes):
        B, K, L, V, dtype = shape
        t, d, tok = _inputs(B, K, L, V, dtype, seed=20 + i)
        inp = (to_torch(t), to_torch(d), to_torch(tok))
        cases.append((shape, inp, [sg.specgbv_verify(*inp, 0.8, 3, 1) for _ in range(2)]))
    torch.cuda.synchronize()

    def read(c, n):
        (B, K, L, V, dtype), _, runs = c
        res = sg.specgbv_read_intermediates(runs[n][3], B, K, L, V, 1 if dtype == "bf16" else 0)
        res.update(out=[x.cpu().numpy().copy() for x in runs[n][:3]])
        return res

    alone = [read(c, 0) for c in cases]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    big, other = torch.empty(1 << 28, dtype=torch.uint8, device="cuda"), torch.empty(1 << 28, dtype=torch.uint8, device="cuda")
    busy = torch.cuda.Stream()
    for _ in range(5):
        with torch.cuda.stream(busy):
            for _ in range(8):
                big.copy_(other)
        for rep in range(4):
            for n, st in enumerate(streams):
                with torch.cuda.stream(st):
                    for _, inp, runs in (cases if (rep + n) % 2 else cases[::-1]):
                        sg.specgbv_verify(*inp, 0.8, 3, 1, workspace=runs[n][3], out=runs[n][:3])
        torch.cuda.synchronize()
        for i, c in enumerate(cases):
            for n in range(2):
                got = read(c, n)
                for key, want in alone[i].items():
                    if key == "out":
                        assert all(np.array_equal(a, b) for a, b in zip(want, got[key])), (c[0], n)
                    else:
                        assert np.array_equal(want, got[key], equal_nan=True), (c[0], n, key)
