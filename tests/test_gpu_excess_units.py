"""Rows whose E = nu^2 (s - g) the final-token kernel's workgroups sum together: a workgroup's waves share a (row, part) unit
by four, by two, or take one each, by how many units there are for a workgroup (needs an MI355X: run with -m gpu)."""
import pytest

import test_gpu_peaked_rows as peaked

pytestmark = pytest.mark.gpu


# 16 or 17 segments: four or five workgroups per prefix.  Marked rows of the two prefixes: two and one (two waves a unit,
# and four); then four and more (one wave a unit), more units than the prefix has waves, and whole rows and ragged ones.
@pytest.mark.parametrize("dtype,V,K,L", [("f32", 8192, 2, 2), ("bf16", 8199, 2, 2), ("bf16", 8200, 2, 3), ("f32", 8193, 3, 5)])
@pytest.mark.parametrize("polls", [None, "0"])
def test_waves_share_units(dtype, V, K, L, polls, monkeypatch):
    if polls is not None:                                   # every workgroup sums every unit itself
        monkeypatch.setenv("SPECGBV_EXCESS_POLLS", polls)
    peaked.test_block_ratio_runs_away("split", dtype, V, 2, K, L)
