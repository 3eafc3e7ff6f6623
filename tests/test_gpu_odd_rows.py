"""Rows that are not a multiple of the 16-byte vector on the two-pass schedule, in Algorithm 2 and under pending
modifications: every remainder, rows of one vector and less (needs an MI355X: run with -m gpu)."""
import numpy as np
import pytest

from parity_util import check_case
from specgbv_synth import Workload, make_inputs
from test_gpu_modification import _check_modify
from test_gpu_pending import check_pending

pytestmark = pytest.mark.gpu

SHAPES = [(V, "bf16") for V in (5, 8, 9, 15, 4097, 4103, 8198)] + [(V, "f32") for V in (3, 4, 5, 7, 2049, 4094, 8199)]


def _inputs(B, K, L, V, dtype):
    t, d, tok = make_inputs(Workload("odd", B, K, L, V, dtype, 2.0, 0.8, head=min(8, V // 2), temperature=0.9), seed=3 + V)
    tok[:, 0, -1] = V - 1                                  # a drafted token in the vector that is not whole
    return t, d, tok


@pytest.mark.parametrize("V,dtype", SHAPES)
def test_two_pass(V, dtype):
    t, d, tok = _inputs(3, 2, 3, V, dtype)
    check_case(t, d, tok, 0.9, 4, 1, "split", "odd rows split %d %s" % (V, dtype))


@pytest.mark.parametrize("V,dtype", SHAPES)
def test_modify(V, dtype):
    t, d, tok = _inputs(2, 3, 3, V, dtype)
    _check_modify(np.ascontiguousarray(t[:, :, :3]), d, tok, 0.9, np.array([0.2, -0.4]), np.array([2, 1], np.int32), "odd rows modify %d %s" % (V, dtype))


@pytest.mark.parametrize("V,dtype", [(49152, "bf16"), (49145, "bf16"), (49153, "bf16"), (4097, "bf16"),
                                     (24576, "f32"), (24573, "f32"), (24577, "f32"), (24580, "f32"), (2049, "f32")])
def test_modify_rows_in_registers(V, dtype):
    """Both sides of the edge between the two tiles (12 and 40 vectors for each of 512 threads), whole vectors and a repeated
    end, and an end of its own slot."""
    test_modify(V, dtype)


@pytest.mark.parametrize("V,dtype", [s for s in SHAPES if s[0] > 100])
def test_pending(V, dtype):
    t, d, tok = _inputs(6, 2, 4, V, dtype)
    rng = np.random.default_rng(V)
    check_pending(t, d, tok, 0.9, 4, 1, rng.normal(0, 0.5, 6), rng.integers(0, 4, 6).astype(np.int32), "odd rows pending %d %s" % (V, dtype))


@pytest.mark.parametrize("algo", ["auto", "split"])
def test_many_drafts_of_short_odd_rows(algo):
    """600 prompts: among so many rows some have nearly equal sums in Eq. (hik), and h then takes ln nu to 2e-7."""
    t, d, tok = make_inputs(Workload("short", 600, 2, 3, 100, "bf16", 2.5, 0.9, head=20, temperature=0.8), seed=5)
    tok[:, 0, -1] = 99
    check_case(t, d, tok, 0.8, 3, 1, algo, "odd rows, 600 prompts")


@pytest.mark.parametrize("V", [515, 2048, 2051, 4099, 8192])
@pytest.mark.parametrize("T", [1.0, 0.7])
def test_modify_in_place(V, T):
    """Float32 results in the buffers of their inputs against results in buffers of their own.  Where the two take kernels that
    add up in another order, a normaliser moves by 1e-6 at most (512 float32 partial sums of up to 2^5 entries), and with it
    the probabilities, relatively; they are compared, not their logarithms, which have a pole where a weight is zero."""
    import torch
    import paper_2604_25925_amd as sg
    from parity_util import to_torch
    B, K, M = 6, 3, 3
    t, d, tok = make_inputs(Workload("place", B, K, M, V, "f32", 2.0, 0.8, head=8, temperature=T), seed=V)
    tl, dl, tk = to_torch(t), to_torch(d), to_torch(tok)
    carry = torch.from_numpy(np.linspace(-0.5, 0.5, B)).cuda()
    count = torch.from_numpy(np.array([0, 1, 2, 3, 3, 2], np.int32)).cuda()
    own = sg.specgbv_modify_target(tl, dl, tk, T, carry, count, want_logp=True, want_norm=True)
    tp, dp = tl.clone(), dl.clone()
    here = sg.specgbv_modify_target(tp, dp, tk, T, carry, count, want_logp=True, want_norm=True, out={"logq": tp, "logp": dp})
    torch.cuda.synchronize()
    assert torch.equal(own["fallback"], here["fallback"])
    assert torch.allclose(own["norm"], here["norm"], rtol=1e-6, atol=1e-9)
    for k in ("logq", "logp"):
        assert torch.allclose(own[k].double().exp(), here[k].double().exp(), rtol=1e-5, atol=1e-8), k
