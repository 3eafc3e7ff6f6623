"""Which schedule a call without a wish gets, where the nearest other one takes a tenth to a third longer (needs an MI355X:
run with -m gpu).  Which one ran is told by what it leaves in the workspace: the rows schedule zeros in the words of its parts, and
each schedule writes in places of its own (the chain's lists of rows)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _runs(B, K, L, V, dtype, algos):
    import torch
    import paper_2604_25925_amd as sg
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V + B)
    ty = torch.bfloat16 if dtype == "bf16" else torch.float32
    t = torch.empty((B, K, L + 1, V), dtype=ty, device="cuda").normal_(0.0, 3.0, generator=gen)
    d = torch.empty((B, K, L, V), dtype=ty, device="cuda").normal_(0.0, 3.0, generator=gen)
    tok = torch.randint(V, (B, K, L), dtype=torch.int32, device="cuda", generator=gen)
    code = 1 if dtype == "bf16" else 0
    out = []
    for algo in algos:
        kept, left = True, []
        for fill in (165, 90):
            ws = torch.full((sg.specgbv_workspace_bytes(B, K, L, V, code),), fill, dtype=torch.uint8, device="cuda")
            sg.specgbv_verify_ex(t, d, tok, 0.8, 3, 1, algo=algo, workspace=ws)
            torch.cuda.synchronize()
            left.append(ws.cpu().numpy())
            kept = kept & (left[-1] == fill)
        res = sg.specgbv_read_intermediates(ws, B, K, L, V, code)
        out.append(_Run(np.stack([res["lse_q"], res["lse_p"]]), ~kept.reshape(-1, 256).all(1), _parts_with_words(left[0], 165, B * K * L)))
    return out


class _Run:
    def __init__(self, normalisers, written, parts):
        # (written: which 256 bytes; by the byte, what a final selection holds beyond its levels may be any value, a filling too.
        # parts: 0 where there are no such words)
        self.normalisers, self.written, self.parts = normalisers, written, parts


def _parts_with_words(ws, fill, rows):
    """How many parts' words (32 bytes each, of the room of 16 parts per row) a call has left zeros in, and in nothing else there."""
    for parts in (1, 2, 4, 8, 16):
        want = np.full((rows, 16, 32), fill, np.uint8)
        want[:, :parts] = 0
        want = want.reshape(-1)
        for o in range(0, len(ws) - want.size + 1, 256):
            if ws[o] == 0 and np.array_equal(ws[o:o + want.size], want):
                return parts
    return 0


@pytest.mark.parametrize("B,K,L,V,dtype", [
    (8, 8, 8, 33000, "bf16"), (8, 4, 8, 66000, "bf16"), (16, 4, 4, 132000, "bf16"),     # parts of 1032 vectors
    (8, 4, 4, 140000, "f32"),                                                          # parts of 2188
    (64, 2, 4, 140000, "f32"),                                                         # rows the chain keeps half of on chip
    (128, 1, 5, 24000, "bf16"), (24, 8, 4, 18000, "bf16"),                              # one round of workgroups and a bit
])
def test_two_passes(B, K, L, V, dtype):
    auto, split = _runs(B, K, L, V, dtype, ("auto", "split"))
    assert np.array_equal(auto.written, split.written) and auto.parts == 0 and split.parts == 0
    assert np.array_equal(auto.normalisers, split.normalisers)


@pytest.mark.parametrize("B,K,L,V,dtype", [
    (8, 8, 8, 65536, "bf16"), (32, 4, 4, 8192, "bf16"), (20, 8, 6, 24000, "bf16"), (8, 4, 5, 32000, "f32"), (1, 3, 8, 128256, "bf16"),
])
def test_rows(B, K, L, V, dtype):
    auto, split = _runs(B, K, L, V, dtype, ("auto", "split"))
    assert auto.parts > 0 and split.parts == 0
    np.testing.assert_allclose(auto.normalisers, split.normalisers, rtol=0, atol=1e-6)         # (2e-7 each)


@pytest.mark.parametrize("B,K,L,V,dtype", [(24, 8, 4, 66000, "bf16"), (64, 8, 2, 32000, "f32")])
def test_chain(B, K, L, V, dtype):
    auto, chain, split = _runs(B, K, L, V, dtype, ("auto", "chain", "split"))
    assert np.array_equal(auto.written, chain.written) and not np.array_equal(auto.written, split.written) and auto.parts == 0
    assert np.array_equal(auto.normalisers, chain.normalisers)
