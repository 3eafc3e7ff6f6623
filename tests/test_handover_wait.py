"""Between the device-scope stores of partial sums and the counter update that announces them the compiled kernels wait for
the stores (a barrier or a workgroup-scope fence alone does not).  Looked for in the assembly hipcc makes of them, along the
paths its branches allow: from such a store no path leads to the counter's atomic, nor to the barrier in front of it (through
which the other waves hand their stores over), without a wait for all of the wave's memory operations."""
import os
import re
import subprocess

import pytest

from paper_2604_25925_amd.build import CSRC, FLAGS, hipcc

WAIT = re.compile(r"s_waitcnt\b.*\bvmcnt\(0\)")


def _kernels(source, tmp_path):
    out = os.path.join(str(tmp_path), "k.s")
    flags = [f for f in FLAGS if f != "-fPIC"]
    subprocess.run([hipcc(), *flags, "-S", "--offload-device-only", os.path.join(CSRC, source), "-o", out], check=True,
                   capture_output=True)
    name, body = None, {}
    for line in open(out):
        line = line.split(";")[0].strip()
        m = re.match(r"^(_Z\S+):", line)
        if m:
            name = m.group(1)
        if line.startswith(".Lfunc_end"):
            name = None
        if name and line and not (line.startswith(".") and not line.endswith(":")):
            body.setdefault(name, []).append(line)
    return body


def _successors(lines):
    at = {s[:-1]: i for i, s in enumerate(lines) if s.endswith(":")}
    nxt = []
    for i, s in enumerate(lines):
        op = s.split()[0]
        assert not op.startswith(("s_setpc", "s_swappc", "s_cbranch_g_fork")), s      # (no calls, no computed branches)
        step = [] if op in ("s_branch", "s_endpgm") else [i + 1]
        if op == "s_branch" or op.startswith("s_cbranch"):
            step.append(at[s.split()[1]])
        nxt.append([j for j in step if j < len(lines)])
    return nxt


def _reach(starts, nxt, stop):
    """Lines that some path from behind `starts` comes to; a path ends at a line for which stop holds."""
    seen, todo = set(), [j for i in starts for j in nxt[i]]
    while todo:
        i = todo.pop()
        if i in seen:
            continue
        seen.add(i)
        if not stop(i):
            todo.extend(nxt[i])
    return seen


def unannounced(lines):
    """(number of counter updates, stores that reach one, or the barrier in front of it, without a wait)."""
    nxt = _successors(lines)
    adds = [i for i, s in enumerate(lines) if s.startswith("global_atomic_add")]
    stores = [i for i, s in enumerate(lines) if s.startswith("global_store") and re.search(r"\bsc1\b", s)]
    barriers = [i for i, s in enumerate(lines) if s.startswith("s_barrier")]
    fronts = {b for b in barriers if any(a in _reach([b], nxt, lambda i: lines[i].startswith("s_barrier")) for a in adds)}
    bad = []
    for st in stores:
        ahead = _reach([st], nxt, lambda i: bool(WAIT.match(lines[i])) or i in fronts or i in adds)
        if any(i in ahead and not WAIT.match(lines[i]) for i in list(fronts) + adds):
            bad.append(st)
    return len(adds), bad, stores


@pytest.mark.parametrize("source,kernel,count", [("specgbv_decide.hip", "k_final", 8), ("specgbv_split.hip", "k_pend_norm", 4)])
def test_counter_updates_wait_for_the_stores_before_them(source, kernel, count, tmp_path):
    if not os.path.exists(hipcc()):
        pytest.skip("no hipcc")
    seen = 0
    for name, lines in _kernels(source, tmp_path).items():
        if kernel not in name:
            continue
        adds, bad, stores = unannounced(lines)
        assert adds and stores, name
        assert not bad, "%s: no wait behind %s" % (name, [lines[i] for i in bad])
        # the same listing without the waits is found out, and so is one whose waits are on another path than the store's
        assert unannounced([s for s in lines if not WAIT.match(s)])[1], name
        away = [t for i, s in enumerate(lines) for t in (("s_cbranch_execz .Lskip%d" % i, s, ".Lskip%d:" % i) if WAIT.match(s) else (s,))]
        assert unannounced(away)[1], name
        seen += adds
    assert seen >= count
