"""K-SEQ rows kept in registers, at the edges of their tiles (16, 32 and 64 entries for each of 512 threads) and with
every remainder of a vector, against the oracle (needs an MI355X: run with -m gpu)."""
import numpy as np
import pytest

import test_gpu_peaked_rows as peaked
from parity_util import to_torch
from specgbv_synth import Workload, f32_to_bf16_bits, make_inputs
from test_gpu_comparison import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K,L,V,dtype", [
    (3, 4, 2, 8, "bf16"), (3, 4, 2, 13, "bf16"), (3, 4, 2, 4, "f32"), (3, 4, 2, 7, "f32"), (3, 4, 2, 3, "f32"),
    (2, 4, 3, 8192, "bf16"), (2, 4, 3, 8193, "bf16"), (2, 4, 3, 8191, "f32"), (2, 4, 3, 8195, "f32"),
    (2, 4, 3, 16384, "bf16"), (2, 4, 3, 16377, "bf16"), (2, 4, 3, 16385, "bf16"), (2, 4, 3, 16382, "f32"), (2, 4, 3, 16385, "f32"),
    (2, 1, 3, 16384, "f32"), (2, 1, 3, 16388, "f32"), (2, 1, 3, 16385, "bf16"), (2, 1, 3, 32765, "bf16"),
    (2, 4, 3, 32768, "bf16"), (2, 4, 3, 32761, "bf16"), (2, 4, 3, 32769, "bf16"), (2, 4, 3, 32766, "f32"), (2, 4, 3, 32772, "f32"),
])
def test_tiles(B, K, L, V, dtype):
    t, d, tok = make_inputs(Workload("kseq", B, K, L, V, dtype, 2.5, 0.8, head=min(8, V // 2), temperature=0.8), seed=3)
    check(t, d, tok, 0.8, 3, 1, None, "K-SEQ tiles %s" % ((B, K, L, V, dtype),), rho_tol=3.0)


@pytest.mark.parametrize("B,L,V,sigma_d,T,seed", [(64, 4, 301, 1.0, 0.4, 5), (64, 3, 100, 0.25, 0.3, 1)])
def test_roots_behind_a_change_of_slope(B, L, V, sigma_d, T, seed):
    """Low temperatures: one entry holds nearly all mass, and the equation for rho turns flat by orders of magnitude as
    rho p passes q there, so that a short Newton step in front of that point says nothing about the root."""
    t, d, tok = make_inputs(Workload("kink", B, 4, L, V, "bf16", 3.0, sigma_d, head=min(50, V // 4), temperature=T), seed=seed)
    check(t, d, tok, T, 1, 1, None, "K-SEQ roots behind a change of slope V=%d" % V)


@pytest.mark.parametrize("V,dtype,T", [(13, "bf16", 0.8), (100, "bf16", 0.8), (1003, "bf16", 0.4), (4095, "bf16", 0.7),
                                       (5, "f32", 1.0), (101, "f32", 0.8), (2047, "f32", 0.7)])
def test_normalisers_of_short_odd_rows(V, dtype, T):
    """Rows that are not a multiple of the vector and give no thread more than one: their normalisers are summed in float64.
    Bound: the scaled logits' scale is float32(log2 e / T) on both sides; a term's exponential is good to 2e-10, the sum
    and the logarithm to 1e-14: 1e-9 in ln Z.  (A float32 sum relative to one reference is off by up to 2.6e-7 here.)"""
    import torch
    import paper_2604_25925_amd as sg
    B, K, L = 40, 4, 3
    t, d, tok = make_inputs(Workload("norm", B, K, L, V, dtype, 3.0, 1.0, head=max(1, min(50, V // 4)), temperature=T), seed=5)
    tl, dl = to_torch(t), to_torch(d)
    ws = sg.specgbv_verify_kseq(tl, dl, to_torch(tok), T, 1, 1)[3]
    torch.cuda.synchronize()
    got = sg.specgbv_read_intermediates(ws, B, K, L, V, 1 if dtype == "bf16" else 0)
    c = float(np.float32(1.4426950408889634 / float(np.float32(T))))
    for z, name in ((tl[:, :, :L], "lse_q"), (dl, "lse_p")):
        y = z.double().cpu() * c
        m = y.amax(-1, keepdim=True)
        ref = (m[..., 0] + torch.log2(torch.exp2(y - m).sum(-1))).numpy() * 0.693147180559945309417
        err = np.abs(got[name] - ref).max()
        assert err <= 1e-9, "%s: off by %.3g" % (name, err)


@pytest.mark.parametrize("V,dtype", [(32768, "bf16"), (3001, "f32")])
@pytest.mark.parametrize("T", [1.0, 0.4])
def test_near_certain_drafted_tokens(V, dtype, T):
    """Rows whose mass sits on the drafted token to within 1e-3 - 1e-6 in either model: the roots balance the other entries'."""
    B, K, L = 5, 4, 4
    t, d, tok = peaked._case(B, K, L, V, T, seed=31)
    rng = np.random.default_rng(32)
    for b in range(B):
        eq, ep = peaked.EPS[b]
        x0 = int(tok[b, 0, 0])
        peaked._set_probability(t[b, 0, 0], x0, T, 1 - eq)
        peaked._set_probability(d[b, 0, 0], x0, T, 1 - ep)
        for k in range(K):
            t[b, k, 0], d[b, k, 0] = t[b, 0, 0], d[b, 0, 0]
            tok[b, k, 0] = x0 if k != 2 else int(rng.integers(0, V))
            for r in range(1, L):
                if k % 2 == 0:
                    peaked._set_probability(t[b, k, r], int(tok[b, k, r]), T, 1 - eq * (r + 1))
                    peaked._set_probability(d[b, k, r], int(tok[b, k, r]), T, 1 - ep / (r + 1))
    if dtype == "bf16":
        t, d = f32_to_bf16_bits(t), f32_to_bf16_bits(d)
    check(t, d, tok, T, 3, 1, None, "K-SEQ near-certain tokens V=%d %s T=%g" % (V, dtype, T))
