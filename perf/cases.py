"""Performance cases: what a program that decodes with this library has it do, over the range it does it in.

Every case goes through the Python binding, on tensors and buffers that the caller keeps between calls (outputs,
workspace, pending state), as a decoding loop would.  Inputs follow the recipe of specgbv_synth (Gaussian logits with a
Zipf-boosted head, a draft that is a noisy copy of the target, draft tokens sampled from the draft, rows that are a
function of the token block in front of them), made on the GPU from the seed.

`exact` is the same computation in 64 bits in plain torch: the acceptance rule as the equations state it, with sums over
the whole vocabulary, no kernels and no base-2 rescaling.

Verifications return accepted lengths, draft indices and tokens, whole numbers that are the same in every correct
implementation except where a uniform falls within the arithmetic's error of a threshold.  Up to 16 prefixes also return
the block ratio that Algorithm 2 continues from; with more prefixes it is left out, because one such tie in the batch
moves that prefix's final token and with it the ratio by a finite amount.
"""
import math

import numpy as np
import torch

import paper_2604_25925_amd as sg
from paper_2604_25925_amd import binding

ELEM = {"f32": (torch.float32, 4), "bf16": (torch.bfloat16, 2)}
DEVICE = "cuda"
LEVELS = binding.MAX_PENDING


def listed():
    return [
        # the smallest call, on the library's built-in scratch memory: nothing but launches and latency
        _case("verify_tiny", "static", 1, 2, 4, 1000, "f32", 1.0, sigma_t=2.0, sigma_d=0.5, head=0),
        # one interactive prompt, the setting of the paper's own experiments (K = 3, L = 8, T = 0.4, batch 1)
        _case("verify_one_prompt", "verify", 1, 3, 8, 128256, "bf16", 0.4, head=200),
        # a small serving batch, float32 logits
        _case("verify_small_batch", "verify", 8, 4, 5, 32000, "f32", 1.0),
        # a full batch of float32 logits whose caller states that a prefix's drafts share their first rows
        _case("verify_f32", "verify", 64, 8, 8, 32000, "f32", 0.8, shared_row0=True),
        # the benchmark's workload: a full batch, large vocabulary, bfloat16
        _case("verify_bf16", "verify", 32, 8, 8, 128256, "bf16", 1.0, head=200),
        # the largest: many drafts of many prefixes, the largest vocabulary, a badly calibrated draft
        _case("verify_largest", "verify", 128, 16, 8, 152064, "bf16", 0.7, sigma_t=3.5, sigma_d=1.5, scale=0.8, head=500),
        # a batch as requests happen to come in: not a power of two
        _case("verify_uneven_batch", "verify", 40, 8, 8, 32000, "bf16", 0.8),
        # an odd vocabulary (tokens were added to it): rows that start at any address
        _case("verify_odd_vocab", "verify", 41, 7, 6, 32003, "bf16", 0.7),
        # one drafting step of that benchmark's batch: a token for each of the 256 drafts
        _case("draft_tokens", "sample", 32, 8, 1, 128256, "bf16", 1.0, head=200),
        # Algorithm 2 written out for the next iteration of that batch
        _case("modify_target", "modify", 32, 8, 8, 128256, "bf16", 1.0, head=200),
        # three iterations of Algorithm 3 from new requests on, its bookkeeping kept on the GPU
        _case("decode_loop", "loop", 8, 4, 8, 128256, "bf16", 1.0, head=200, iterations=3),
        # the comparison verifier on a batch (SpecTr's K-SEQ rule)
        _case("verify_kseq", "kseq", 32, 4, 8, 32000, "f32", 0.8),
    ]


def _case(name, op, batch, K, L, V, dtype, temperature, sigma_t=3.0, sigma_d=1.0, scale=1.0, head=50, shared_row0=False,
          levels=0, iterations=1):
    c = {"op": op, "batch": batch, "K": K, "L": L, "V": V, "dtype": dtype, "temperature": temperature, "sigma_t": sigma_t,
         "sigma_d": sigma_d, "scale": scale, "head": head, "shared_row0": shared_row0, "levels": levels, "iterations": iterations}
    return dict(c, name=name) if name else c


def draw(rng):
    """Any operation at sizes between the tiny and the largest listed case; no dearer than a tenth of the largest."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["verify", "verify", "verify", "verify", "pending", "loop", "modify", "sample", "kseq"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    V = log_int(1000, 152064)
    V -= V % rng.choice([1, 2, 8, 64, 64])              # any vocabulary size; most are a multiple of something
    K = rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 8, 16])
    L = rng.choice([3, 4, 5, 6, 8, 8, 12])
    batch = log_int(1, 128)
    iterations = 2 if op == "loop" else 1
    entries = 250_000_000 // {"kseq": 4, "modify": 2, "loop": 4, "pending": 2}.get(op, 1)
    while batch > 1 and batch * K * (1 if op == "sample" else L) * V > entries:
        batch = (batch + 1) // 2
    return _case(None, op, batch, K, 1 if op == "sample" else L, V, dtype, rng.choice([0.4, 0.7, 0.8, 1.0, 1.0]),
                 sigma_t=rng.choice([2.0, 3.0, 3.5]), sigma_d=rng.choice([0.25, 1.0, 1.5, 2.0]), scale=rng.choice([0.8, 1.0]),
                 head=0 if V < 2000 else rng.choice([50, 200, 500]), shared_row0=op == "verify" and rng.random() < 0.3,
                 levels=rng.randint(1, 3) if op == "pending" else 0, iterations=iterations)


# ------------------------------------------------------------------------------------------------------------- inputs


def _make_inputs(case, seed):
    """(target [B, K, L+1, V], draft [B, K, L, V], tokens [B, K, L] int32) for the seed."""
    B, K, L, V = (case[k] for k in ("batch", "K", "L", "V"))
    dtype, _ = ELEM[case["dtype"]]
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed) * 1000003 + 17)
    target = torch.empty((B, K, L + 1, V), dtype=dtype, device=DEVICE)
    draft = torch.empty((B, K, L, V), dtype=dtype, device=DEVICE)
    tokens = torch.empty((B, K, L), dtype=torch.int32, device=DEVICE)
    head = min(case["head"], V)
    boost = (6.0 - 1.1 * torch.log(torch.arange(1, head + 1, dtype=torch.float32, device=DEVICE))) if head else None
    T = float(np.float32(case["temperature"]))
    per = max(1, 200_000_000 // (K * V))                # prefixes at a time
    for b0 in range(0, B, per):
        n = min(per, B - b0)
        same = torch.ones((n, K, K), dtype=torch.bool, device=DEVICE)       # drafts that share their first r tokens
        for r in range(L + 1):
            lead = same.to(torch.int8).argmax(dim=2)                        # the first draft with this draft's block
            rows = torch.arange(n, device=DEVICE)[:, None].expand(n, K)
            zq = torch.empty((n, K, V), dtype=torch.float32, device=DEVICE).normal_(0.0, case["sigma_t"], generator=gen)
            if head:
                ids = torch.randint(V, (n, K, head), device=DEVICE, generator=gen)
                zq.scatter_add_(2, ids, boost.expand(n, K, head))
            q = zq.to(dtype)[rows, lead]
            target[b0:b0 + n, :, r] = q
            if r == L:
                break
            noise = torch.empty((n, K, V), dtype=torch.float32, device=DEVICE).normal_(0.0, case["sigma_d"], generator=gen)
            p = noise.add_(zq, alpha=case["scale"]).to(dtype)[rows, lead]
            draft[b0:b0 + n, :, r] = p
            gumbel = zq.exponential_(generator=gen).log_().neg_()
            tok = gumbel.add_(p.float(), alpha=1.0 / T).argmax(dim=2)
            tokens[b0:b0 + n, :, r] = tok.to(torch.int32)
            same &= tok[:, :, None] == tok[:, None, :]
    return target, draft, tokens


def _levels(case, seed):
    """Pending modifications as earlier iterations leave them: ratios near one, counts that shrink with age."""
    r = np.random.RandomState((int(seed) * 7919 + 5) % (1 << 31))
    B, L, n = case["batch"], case["L"], max(1, case["levels"])
    carry = r.normal(0.0, 1.0, (n, B))
    count = np.sort(r.randint(0, L, (n, B)), axis=0).astype(np.int32)
    return carry, count


def _outputs(B, L):
    return (torch.empty(B, dtype=torch.int32, device=DEVICE), torch.empty(B, dtype=torch.int32, device=DEVICE),
            torch.empty((B, L + 1), dtype=torch.int32, device=DEVICE))


def prepare(case, seed):
    B, K, L, V, op = (case[k] for k in ("batch", "K", "L", "V", "op"))
    dt = binding.BF16 if case["dtype"] == "bf16" else binding.F32
    s = {"case": case, "seed": int(seed) & 0x7FFFFFFF}
    if op == "sample":
        s["logits"] = _make_inputs(case, seed)[1].reshape(B * K, V).clone()
        s["out"] = torch.empty(B * K, dtype=torch.int32, device=DEVICE)
        s["workspace"] = torch.empty(max(256, sg.specgbv_sample_workspace_bytes(B * K, V)), dtype=torch.uint8, device=DEVICE)
        return s
    s["inputs"] = [_make_inputs(case, seed + 7 * i) for i in range(case["iterations"])]
    if op == "modify":
        carry, count = _levels(case, seed)
        s["carry"], s["count"] = torch.from_numpy(carry[0]).to(DEVICE), torch.from_numpy(count[0]).to(DEVICE)
        s["out"] = {"logq": torch.empty((B, K, L + 1, V), dtype=torch.float32, device=DEVICE),
                    "logp": torch.empty((B, K, L, V), dtype=torch.float32, device=DEVICE),
                    "norm": torch.empty((B, K, L), dtype=torch.float64, device=DEVICE),
                    "fallback": torch.empty((B, K, L), dtype=torch.int32, device=DEVICE),
                    "workspace": torch.empty(max(256, sg.specgbv_modify_workspace_bytes(B, K, L, 1)), dtype=torch.uint8,
                                             device=DEVICE)}
        return s
    s["outs"] = [_outputs(B, L) for _ in s["inputs"]]
    if op == "static":
        return s
    ws = torch.empty(max(256, sg.specgbv_workspace_bytes(B, K, L, V, dt)), dtype=torch.uint8, device=DEVICE)
    s["workspace"] = ws
    if op == "pending":
        carry, count = _levels(case, seed)
        s["pending"] = (torch.from_numpy(carry).to(DEVICE), torch.from_numpy(count).to(DEVICE))
    if op == "loop":
        s["state"] = torch.empty(sg.specgbv_pending_state_bytes(B), dtype=torch.uint8, device=DEVICE)
        n = LEVELS * B
        s["state_carry"] = s["state"][:n * 8].view(torch.float64).view(LEVELS, B)
        s["state_count"] = s["state"][n * 8:n * 12].view(torch.int32).view(LEVELS, B)
    elif op in ("verify", "pending") and B <= 16:       # the two values the next iteration takes from the workspace
        a, b = sg.specgbv_workspace_carry(ws, B, K, L, V)
        a, b = a - ws.data_ptr(), b - ws.data_ptr()
        s["next"] = (ws[a:a + 8 * B].view(torch.float64), ws[b:b + 4 * B].view(torch.int32))
    return s


def run(s):
    case, seed = s["case"], s["seed"]
    op, T = case["op"], case["temperature"]
    if op == "sample":
        sg.specgbv_sample_tokens(s["logits"], T, seed, 1, 3, out=s["out"], workspace=s["workspace"])
        return {"tokens": s["out"]}
    target, draft, tokens = s["inputs"][0]
    if op == "modify":
        res = sg.specgbv_modify_target(target, draft, tokens, T, s["carry"], s["count"], want_logp=True, want_norm=True,
                                       out=s["out"])
        return {k: res[k] for k in ("logq", "logp", "norm", "fallback")}
    out = s["outs"][0]
    if op == "static":
        sg.specgbv_verify_static(target, draft, tokens, T, seed, 1, out=out)
    elif op == "kseq":
        sg.specgbv_verify_kseq(target, draft, tokens, T, seed, 1, workspace=s["workspace"], out=out)
    elif op == "loop":
        s["state"].zero_()
        for i, ((t, d, k), o) in enumerate(zip(s["inputs"], s["outs"])):
            sg.specgbv_verify_ex(t, d, k, T, seed, 1 + i, workspace=s["workspace"], out=o, pending_state=s["state"])
        return {"steps": [_named(o) for o in s["outs"]], "carry": s["state_carry"], "count": s["state_count"]}
    elif op == "pending":
        sg.specgbv_verify_ex(target, draft, tokens, T, seed, 1, workspace=s["workspace"], out=out, pending=s["pending"])
    elif case["shared_row0"]:
        sg.specgbv_verify_ex(target, draft, tokens, T, seed, 1, workspace=s["workspace"], out=out, shared_row0=True)
    else:
        sg.specgbv_verify(target, draft, tokens, T, seed, 1, workspace=s["workspace"], out=out)
    got = _named(out)
    if "next" in s:
        got["carry"], got["count"] = s["next"]
    return got


def _named(out):
    return {"accepted_len": out[0], "accepted_draft_idx": out[1], "out_tokens": out[2]}


def work(case):
    """Every (target, draft) row pair once, the drafted tokens, the outputs.  Operations for each entry pair: two
    exponentials and two sums for the normalisers, two exponentials, the ratio's subtraction, its power and the sum."""
    B, K, L, V, op = (case[k] for k in ("batch", "K", "L", "V", "op"))
    esz = ELEM[case["dtype"]][1]
    if op == "sample":
        return {"bytes": B * K * (V * esz + 4), "flops": 4 * B * K * V}
    pairs = B * K * L
    if op == "modify":
        rows = B * K * (2 * L + 1)
        return {"bytes": rows * V * (esz + 4) + pairs * 16, "flops": 6 * rows * V}
    if case["shared_row0"]:
        pairs = B * (K * (L - 1) + 1)
    n = case["iterations"]
    return {"bytes": n * (pairs * V * 2 * esz + B * K * L * 4 + B * (L + 3) * 4), "flops": n * 20 * pairs * V}


def tolerance(case):
    """Whole numbers: the odd tie.  Measured against `exact`: block ratios (sums of log-probabilities, 64-bit sums of
    32-bit partial sums) are 1e-8 - 2e-7 off; ln q_new of entries next to ratio one (K ln (1 - ratio), the ratio a 32-bit
    exponential) is what the 1e-5 - 2e-5 of a modification come from, its other outputs are 1e-8 - 4e-8 off."""
    if case["op"] in ("verify", "pending", "loop"):
        return {"rel": 2e-6, "differ": 0.01}
    if case["op"] == "modify":
        return {"rel": 8e-5, "max": 0.05, "differ": 0.001}
    return {"rel": 0.0, "differ": 0.01}


# ---------------------------------------------------------------------------------------------------------- in 64 bits


def _uniforms(seed, offset, prefix, slots):
    """Philox4x32-10 word 0 of (key = seed; counter = offset low, offset high, prefix, slot), as u = (word >> 8) 2^-24."""
    c = [np.full(len(slots), v & 0xFFFFFFFF, np.uint64) for v in (offset, offset >> 32, prefix)] + [np.asarray(slots, np.uint64)]
    k0, k1, low = seed & 0xFFFFFFFF, seed >> 32, np.uint64(0xFFFFFFFF)
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & low, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & low]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return (c[0] >> np.uint64(8)).astype(np.float64) / 16777216.0


def _log_probs(logits, T):
    return torch.log_softmax(logits.double() / float(np.float32(T)), dim=-1)


def _at(rows, tokens):
    return rows.gather(-1, tokens.long().unsqueeze(-1)).squeeze(-1)


def _residual(lq, lp, log_nu, K):
    """q max(1 - p / (nu q), 0)^K over the last dimension (q = 0: 0)."""
    ratio = torch.exp(torch.where(lq > -math.inf, lp - lq - log_nu, math.inf))
    return torch.exp(lq) * (1.0 - ratio).clamp_(min=0.0) ** K


def _modified(lq, lp, tokens, carry, count, K):
    """Algorithm 2 on the rows r < count of every draft: (new rows, their normalisers, where all weights were zero)."""
    M = lp.shape[1]
    step = _at(lq[:, :M], tokens) - _at(lp, tokens)
    new, norm, zero = lq.clone(), torch.ones_like(step), torch.zeros_like(step, dtype=torch.int32)
    for r in range(min(count, M)):
        log_mu = carry + step[:, :r].sum(dim=1, keepdim=True)
        w = _residual(lq[:, r], lp[:, r], log_mu, K)
        W = w.sum(dim=1, keepdim=True)
        new[:, r] = torch.where(W > 0, torch.log(w / W), lq[:, r])
        norm[:, r], zero[:, r] = torch.where(W > 0, W, 1.0).squeeze(1), (W <= 0).int().squeeze(1)
    return new, norm, zero


def _draw_token(w, u):
    """First index whose running sum exceeds u times the total."""
    cum = torch.cumsum(w, dim=0)
    i = int(torch.searchsorted(cum, u * cum[-1], right=True))
    return min(i, int(w.nonzero()[-1]))


def _decide(lq, lp, tokens, seed, offset, b):
    """Algorithm 1 for one prefix from log-probability rows lq [K, L+1, V], lp [K, L, V].
    (tau, f, emitted tokens, log block ratio behind the final token)"""
    K, L, V = lp.shape
    tq, tp = _at(lq[:, :L], tokens), _at(lp, tokens)
    log_nu, log_P = torch.cumsum(tq - tp, dim=1), torch.cumsum(tp, dim=1)
    nu, P, inv = torch.exp(log_nu), torch.exp(log_P), torch.exp(-log_nu)
    g = (1.0 - inv).clamp(min=0.0) ** K
    cK = -torch.expm1(K * torch.log1p(-P)) / P
    h = nu * (1.0 - g) / cK                                             # whole blocks, Eq. (hLk), and then Eq. (hik)
    for i in range(1, L):
        s = _residual(lq[:, i], lp[:, i], log_nu[:, i - 1:i], K).sum(dim=1)
        num, den = nu[:, i - 1] * (s - g[:, i - 1]), cK[:, i - 1] - nu[:, i - 1] * (1.0 - s)
        h[:, i - 1] = torch.where(den > 0, num / den, 1.0)
    h = torch.nan_to_num(h, nan=0.0).clamp_(0.0, 1.0).cpu().numpy()
    u = _uniforms(seed, offset, b, np.arange(K * L + 1))
    toks, rejected, tau, f = tokens.cpu().numpy(), set(), 0, -1
    for k in range(K):
        start = tau
        for i in range(start + 1, L + 1):
            block = tuple(toks[k, :i])
            if block in rejected:
                continue
            if u[k * L + i - 1] < h[k, i - 1]:
                tau, f = i, k
            else:
                rejected.add(block)
        if tau == L:
            break
    kf = max(f, 0)
    if tau == L:
        y, carry = _draw_token(torch.exp(lq[kf, L]), u[K * L]), 0.0
    else:
        ln = float(log_nu[kf, tau - 1]) if tau else 0.0
        w = _residual(lq[kf, tau], lp[kf, tau], ln, K)
        y = _draw_token(w if float(w.sum()) > 0 else torch.exp(lq[kf, tau]), u[K * L])
        carry = ln + float(lq[kf, tau, y] - lp[kf, tau, y])
    return tau, f, [int(t) for t in toks[kf, :tau]] + [y], carry


def _decide_kseq(lq, lp, tokens, seed, offset, b):
    """The K-SEQ rule for one prefix: (tau, lead draft or -1, emitted tokens)."""
    K, L, V = lp.shape
    u = _uniforms(seed, offset, b, np.arange(K * L + 1))
    toks, alive, kept = tokens.cpu().numpy(), list(range(K)), []
    for i in range(L):
        lead, n = alive[0], len(alive)
        q, p = torch.exp(lq[lead, i]), torch.exp(lp[lead, i])
        lo, hi = 1.0, float(n)
        for _ in range(60 if n > 1 else 0):
            mid = 0.5 * (lo + hi)
            G = float(torch.minimum(mid * p, q).sum())
            lo, hi = (lo, mid) if G - 1.0 + (1.0 - min(G / mid, 1.0)) ** n >= 0 else (mid, hi)
        rho = 0.5 * (lo + hi) if n > 1 else 1.0
        won = [j for j in alive if u[j * L + i] < float(q[int(toks[j, i])] / (rho * p[int(toks[j, i])]))]
        if not won:
            w = (q - rho * p).clamp_(min=0.0)
            return i, lead if i else -1, kept + [_draw_token(w if float(w.sum()) > 0 else q, u[K * L])]
        kept.append(int(toks[won[0], i]))
        alive = [j for j in alive if toks[j, i] == kept[-1]]
    return L, alive[0], kept + [_draw_token(torch.exp(lq[alive[0], L]), u[K * L])]


def _stacked(rows, L, like):
    """Per prefix (tau, f, emitted tokens) as the three output tensors."""
    out = np.full((len(rows), L + 1), -1, np.int32)
    for b, r in enumerate(rows):
        out[b, :len(r[2])] = r[2]
    ints = [np.array([r[j] for r in rows], np.int32) for j in (0, 1)]
    return {"accepted_len": ints[0], "accepted_draft_idx": ints[1], "out_tokens": out}


def exact(case, seed):
    B, K, L, V, op, T = (case[k] for k in ("batch", "K", "L", "V", "op", "temperature"))
    s = int(seed) & 0x7FFFFFFF
    if op == "sample":
        logits = _make_inputs(case, seed)[1].reshape(B * K, V)
        u = [_uniforms(s, 1, r, [(1 << 31) + 3])[0] for r in range(B * K)]
        return {"tokens": np.array([_draw_token(torch.exp(_log_probs(logits[r], T)), u[r]) for r in range(B * K)], np.int32)}
    sets = [_make_inputs(case, seed + 7 * i) for i in range(case["iterations"])]
    target, draft, tokens = sets[0]
    if op == "modify":
        carry, count = _levels(case, seed)
        res = {"logq": torch.empty(target.shape, dtype=torch.float64, device=DEVICE),
               "logp": torch.empty(draft.shape, dtype=torch.float64, device=DEVICE),
               "norm": torch.empty((B, K, L), dtype=torch.float64, device=DEVICE),
               "fallback": torch.empty((B, K, L), dtype=torch.int32, device=DEVICE)}
        for b in range(B):
            lq, lp = _log_probs(target[b], T), _log_probs(draft[b], T)
            res["logp"][b] = lp
            res["logq"][b], res["norm"][b], res["fallback"][b] = _modified(lq, lp, tokens[b], float(carry[0, b]), int(count[0, b]), K)
        return res
    if op == "kseq":
        return _stacked([_decide_kseq(_log_probs(target[b], T), _log_probs(draft[b], T), tokens[b], s, 1, b) for b in range(B)], L, target)
    if op == "loop":
        return _exact_loop(case, sets, s)
    levels = _levels(case, seed) if op == "pending" else (np.zeros((0, B)), np.zeros((0, B), np.int32))
    rows = []
    for b in range(B):
        lq, lp = _log_probs(target[b], T), _log_probs(draft[b], T)
        if case["shared_row0"]:
            lq[:, 0], lp[:, 0] = lq[0, 0].clone(), lp[0, 0].clone()
        for carry, count in zip(*levels):
            lq = _modified(lq, lp, tokens[b], float(carry[b]), int(count[b]), K)[0]
        rows.append(_decide(lq, lp, tokens[b], s, 1, b))
    got = _stacked(rows, L, target)
    if op != "static" and B <= 16:
        got["carry"] = np.array([r[3] for r in rows])
        got["count"] = np.array([L - r[0] - 1 if r[0] < L else 0 for r in rows], np.int32)
    return got


def _exact_loop(case, sets, s):
    B, K, L, T = (case[k] for k in ("batch", "K", "L", "temperature"))
    carries, counts = np.zeros((LEVELS, B)), np.zeros((LEVELS, B), np.int32)
    steps = [[] for _ in sets]
    for b in range(B):
        levels = []                                                     # (log ratio, rows left), oldest first
        for i, (target, draft, tokens) in enumerate(sets):
            lq, lp = _log_probs(target[b], T), _log_probs(draft[b], T)
            under = [lq]
            for carry, count in levels:
                under.append(_modified(under[-1], lp, tokens[b], carry, count, K)[0])
            tau, f, emitted, carry_new = _decide(under[-1], lp, tokens[b], s, 1 + i, b)
            steps[i].append((tau, f, emitted))
            kf, moved = max(f, 0), []
            for (carry, count), rows in zip(levels, under):             # each along the emitted tokens, under its own rows
                if tau < L and count > tau + 1:
                    gain = sum(float(rows[kf, j, e] - lp[kf, j, e]) for j, e in enumerate(emitted))
                    moved.append((carry + gain, count - (tau + 1)))
            levels = moved + ([(carry_new, L - tau - 1)] if tau < L - 1 else [])
        for j, (carry, count) in enumerate(levels):
            carries[j, b], counts[j, b] = carry, count
    return {"steps": [_stacked(r, L, None) for r in steps], "carry": carries, "count": counts}
