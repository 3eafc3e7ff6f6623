"""Error of the level passes' normalisers, whose rows are shared among workgroups and summed in float32, against 64 bits (needs an
MI355X: run with -m gpu)."""
import numpy as np
import pytest

from parity_util import run_gpu

pytestmark = pytest.mark.gpu


def _temperature():
    """A temperature whose scale log2(e) / T is a float32 value to 1e-11, so that the weights' scale is not an error of its own."""
    t = np.arange(1 << 16).astype(np.uint32) + np.float32(1.4).view(np.uint32)
    x = np.log2(np.e) / t.view(np.float32).astype(np.float64)
    rel = np.abs(x.astype(np.float32).astype(np.float64) / x - 1.0)
    assert rel.min() < 1e-11
    return t.view(np.float32)[rel.argmin()]


def _summed_term_by_term(z, c, parts, per_vec):
    """Relative error of a row's float32 sum as `parts` workgroups of 512 threads make it, each thread term after term."""
    l = np.log2(np.exp2(z.astype(np.float64) * c).sum())
    w = np.exp2(z * np.float32(c) - np.float32(l)).astype(np.float32)
    v = w.reshape(-1, per_vec)
    per = -(-len(v) // parts)
    total = 0.0
    for p in range(parts):
        x = v[p * per:(p + 1) * per]
        steps = -(-len(x) // 512)
        x = np.concatenate([x, np.zeros((steps * 512 - len(x), per_vec), np.float32)]).reshape(steps, 512, per_vec)
        acc = np.zeros(512, np.float32)
        for s in range(steps):
            for j in range(per_vec):
                acc = acc + x[s, :, j]
        total += acc.astype(np.float64).sum()
    return total / w.astype(np.float64).sum() - 1.0


def test_normalisers():
    """bfloat16 rows of 131072 entries; in float32, with half as many entries per vector, the weights' own rounding covers the sum's.
    16 x 2 drafts whose level modifies three rows each, 96 rows: no more error than where four workgroups per compute unit share
    them (ten a row), each thread adding up its entries one by one.  The draft's mass lies where the target has none, so that every
    factor of the modification is one to float32 and the normaliser the row's plain sum; what ln nu is off by, row by row, is that
    sum's error.  1.25: two root mean squares of 96 rows each scatter by 7 %, their ratio by 10 %."""
    B, K, L, V = 16, 2, 4, 131072
    T = float(_temperature())
    c = float(np.float32(np.log2(np.e) / T))
    r = np.random.RandomState(4)
    t = r.normal(0.0, 1.0, (B, K, L + 1, V)).astype(np.float32)
    t = (t.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)
    tok = r.randint(0, V // 2, (B, K, L)).astype(np.int32)
    d = np.full((B, K, L, V), -np.inf, np.float32)
    t[..., V - 1] = -np.inf
    d[..., V - 1] = 0.0
    np.put_along_axis(d, tok[..., None].astype(np.int64), -100.0, axis=3)
    as_bf16 = lambda x: (x.view(np.uint32) >> 16).astype(np.uint16)
    got = run_gpu(as_bf16(t), as_bf16(d), tok, T, 1, 0, pending=(np.zeros(B), np.full(B, 3, np.int32)))["log_nu"].reshape(B, K, L)
    err, old = [], []
    for b in range(B):
        for k in range(K):
            for j in range(3):
                z = t[b, k, j].astype(np.float64) / T
                ln_q = z[tok[b, k, j]] - np.log(np.exp(z).sum())
                ln_p = -100.0 / T - np.log1p(np.exp(-100.0 / T))
                err.append(got[b, k, j] - (got[b, k, j - 1] if j else 0.0) - (ln_q - ln_p))
                old.append(_summed_term_by_term(t[b, k, j], c, 10, 8))
    rms, rms_old = (float(np.sqrt(np.mean(np.square(x)))) for x in (err, old))
    print("rms error of the normalisers %.2e, term by term in ten parts %.2e" % (rms, rms_old))
    assert rms <= 1.25 * rms_old
