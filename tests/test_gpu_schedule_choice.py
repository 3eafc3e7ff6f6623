"""Which schedule a call without a wish gets, where the nearest other one takes a tenth to a third longer (needs an MI355X:
run with -m gpu).  The schedules add their sums up in different orders, so the bits of the rows' normalisers tell them apart."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _normalisers(B, K, L, V, dtype, algos):
    import torch
    import paper_2604_25925_amd as sg
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V + B)
    ty = torch.bfloat16 if dtype == "bf16" else torch.float32
    t = torch.empty((B, K, L + 1, V), dtype=ty, device="cuda").normal_(0.0, 3.0, generator=gen)
    d = torch.empty((B, K, L, V), dtype=ty, device="cuda").normal_(0.0, 3.0, generator=gen)
    tok = torch.randint(V, (B, K, L), dtype=torch.int32, device="cuda", generator=gen)
    out = []
    for algo in algos:
        ws = sg.specgbv_verify_ex(t, d, tok, 0.8, 3, 1, algo=algo)[3]
        torch.cuda.synchronize()
        res = sg.specgbv_read_intermediates(ws, B, K, L, V, 1 if dtype == "bf16" else 0)
        out.append(np.stack([res["lse_q"], res["lse_p"]]))
    return out


@pytest.mark.parametrize("B,K,L,V,dtype", [
    (8, 8, 8, 33000, "bf16"), (8, 4, 8, 66000, "bf16"), (16, 4, 4, 132000, "bf16"),     # parts of 1032 vectors
    (8, 4, 4, 140000, "f32"),                                                          # parts of 2188
    (64, 2, 4, 140000, "f32"),                                                         # rows the chain keeps half of on chip
    (128, 1, 5, 24000, "bf16"), (24, 8, 4, 18000, "bf16"),                              # one round of workgroups and a bit
])
def test_two_passes(B, K, L, V, dtype):
    auto, split = _normalisers(B, K, L, V, dtype, ("auto", "split"))
    assert np.array_equal(auto, split)


@pytest.mark.parametrize("B,K,L,V,dtype", [
    (8, 8, 8, 65536, "bf16"), (32, 4, 4, 8192, "bf16"), (20, 8, 6, 24000, "bf16"), (8, 4, 5, 32000, "f32"), (1, 3, 8, 128256, "bf16"),
])
def test_rows(B, K, L, V, dtype):
    auto, split = _normalisers(B, K, L, V, dtype, ("auto", "split"))
    np.testing.assert_allclose(auto, split, rtol=0, atol=1e-6)         # (2e-7 each)
    # (parts, or the logarithm that ends a row, differ in some rows)
    assert not np.array_equal(auto, split)


@pytest.mark.parametrize("B,K,L,V,dtype", [(24, 8, 4, 66000, "bf16"), (64, 8, 2, 32000, "f32")])
def test_chain(B, K, L, V, dtype):
    auto, chain, split = _normalisers(B, K, L, V, dtype, ("auto", "chain", "split"))
    assert np.array_equal(auto, chain) and not np.array_equal(auto, split)
