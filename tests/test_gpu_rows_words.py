"""The words through which the rows schedule's workgroups hand over normalisers, with whatever the workspace held before a call:
fillings, words of earlier calls of the same and of another shape, and of the same call's earlier replay (needs an MI355X: run
with -m gpu)."""
import numpy as np
import pytest

from parity_util import to_torch
from specgbv_synth import Workload, make_inputs

pytestmark = pytest.mark.gpu

# batch, K, L, V, type; in 8, 16, 1, 4, 8 and 1 parts, of 512, 1094, 750, 563, 1719 and 2125 vectors: each of the four tiles
SHAPES = [(2, 3, 5, 32768, "bf16"), (1, 2, 4, 70001, "f32"), (40, 4, 3, 6000, "bf16"), (3, 2, 1, 9000, "f32"),
          (3, 3, 4, 110000, "bf16"), (18, 3, 5, 8500, "f32")]
PARTS = [8, 16, 1, 4, 8, 1]


class _Calls:
    def __init__(self, shape, ws=None):
        import torch
        import paper_2604_25925_amd as sg
        B, K, L, V, dtype = shape
        self.dims = (B, K, L, V, 1 if dtype == "bf16" else 0)
        w = Workload("words", B, K, L, V, dtype, 2.5, 0.9, head=20, temperature=0.8)
        self.sets = [[to_torch(a) for a in make_inputs(w, seed=s)] for s in (5, 6)]
        self.bufs = [a.clone() for a in self.sets[0]]
        n = sg.specgbv_workspace_bytes(B, K, L, V, self.dims[4])
        self.ws = torch.zeros(n, dtype=torch.uint8, device="cuda") if ws is None else ws[:n]
        self.out = (torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty(B, dtype=torch.int32, device="cuda"),
                    torch.empty((B, L + 1), dtype=torch.int32, device="cuda"))

    def load(self, i):
        for b, a in zip(self.bufs, self.sets[i]):
            b.copy_(a)

    def call(self):
        import paper_2604_25925_amd as sg
        sg.specgbv_verify(*self.bufs, 0.8, 9, 1, workspace=self.ws, out=self.out)

    def results(self):
        import torch
        import paper_2604_25925_amd as sg
        torch.cuda.synchronize()
        res = sg.specgbv_read_intermediates(self.ws, *self.dims)
        return [t.cpu().numpy() for t in self.out] + [res[k] for k in ("lse_q", "lse_p", "log_nu", "s", "h")]


def _same(a, b):
    return all(np.array_equal(x, y, equal_nan=True) for x, y in zip(a, b))


@pytest.mark.parametrize("shape,parts", zip(SHAPES, PARTS))
def test_words_are_used_and_cleared(shape, parts):
    """In a workspace full of one byte, a call leaves zeros in exactly the words of its parts (32 bytes each, of the room of 16
    parts per row): the shapes above go to the rows schedule in the parts that the other tests count on, and a replay with the
    same number finds none of the words."""
    import torch
    c = _Calls(shape)
    c.ws.fill_(165)
    c.call()
    torch.cuda.synchronize()
    rows = shape[0] * shape[1] * shape[2]
    ws = c.ws.cpu().numpy()
    want = np.full((rows, 16, 32), 165, np.uint8)
    want[:, :parts] = 0
    want = want.reshape(-1)
    at = [o for o in range(0, len(ws) - want.size + 1, 256) if ws[o] == 0 and np.array_equal(ws[o:o + want.size], want)]
    assert at, "no such words"


@pytest.mark.parametrize("shape", SHAPES)
def test_whatever_the_workspace_held(shape):
    import torch
    c = _Calls(shape)
    want = []
    for i in (0, 1):
        c.load(i)
        c.ws.zero_()
        c.call()
        want.append(c.results())
    assert not _same(*want)
    for n in range(6):
        if n in (1, 2):
            c.ws.fill_(255 if n == 1 else 0)
        if n == 3:
            c.ws.random_(0, 256)
        c.load(n & 1)                                       # (n = 0, 4, 5: behind a call with other inputs)
        c.call()
        assert _same(c.results(), want[n & 1]), n


def test_two_shapes_in_one_workspace():
    import torch
    import paper_2604_25925_amd as sg
    sizes = [sg.specgbv_workspace_bytes(s[0], s[1], s[2], s[3], 1 if s[4] == "bf16" else 0) for s in SHAPES[:3]]
    ws = torch.zeros(max(sizes), dtype=torch.uint8, device="cuda")
    calls = [_Calls(s, ws) for s in SHAPES[:3]]
    want = []
    for c in calls:
        ws.zero_()
        c.call()
        want.append(c.results())
    for n in (0, 1, 2, 1, 0, 2, 2, 0):
        calls[n].call()
        assert _same(calls[n].results(), want[n]), n


@pytest.mark.parametrize("shape", SHAPES)
def test_replays_on_other_inputs(shape):
    import torch
    c = _Calls(shape)
    want = []
    for i in (0, 1):
        c.load(i)
        c.call()
        want.append(c.results())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        c.call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c.call()
    for n in range(6):
        c.load(n & 1)
        if n == 4:
            c.call()                                        # an eager call between replays
        torch.cuda.synchronize()
        graph.replay()
        assert _same(c.results(), want[n & 1]), n
