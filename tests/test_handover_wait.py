"""Between the device-scope stores of partial sums and the counter update that announces them the compiled kernels wait
for the stores (a barrier or a workgroup-scope fence alone does not): looked for in the assembly hipcc makes of them."""
import os
import re
import subprocess

import pytest

from paper_2604_25925_amd.build import CSRC, FLAGS, hipcc


def _kernels(source, tmp_path):
    out = os.path.join(str(tmp_path), "k.s")
    flags = [f for f in FLAGS if f != "-fPIC"]
    subprocess.run([hipcc(), *flags, "-S", "--offload-device-only", os.path.join(CSRC, source), "-o", out], check=True,
                   capture_output=True)
    name, body = None, {}
    for line in open(out):
        m = re.match(r"^(_Z\S+):", line)
        if m:
            name = m.group(1)
        if name:
            body.setdefault(name, []).append(line.strip())
    return body


@pytest.mark.parametrize("source,kernel,count", [("specgbv_decide.hip", "k_final", 4), ("specgbv_split.hip", "k_pend_norm", 4)])
def test_counter_updates_wait_for_the_stores_before_them(source, kernel, count, tmp_path):
    if not os.path.exists(hipcc()):
        pytest.skip("no hipcc")
    seen = 0
    for name, lines in _kernels(source, tmp_path).items():
        if kernel not in name:
            continue
        adds = [i for i, s in enumerate(lines) if s.startswith("global_atomic_add")]
        stores = [i for i, s in enumerate(lines) if s.startswith("global_store") and " sc1" in s]
        assert adds and stores, name
        for a in adds:
            last = max(i for i in stores if i < a)
            assert any(re.match(r"s_waitcnt vmcnt\(0\)", s) for s in lines[last:a]), "%s: no wait in front of line %d" % (name, a)
            seen += 1
    assert seen >= count
