"""bench.py's figures that come from committed counter summaries."""

import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("n,workload", [(6000, "n6000"), (16000, "n16000")])
def test_counted_figures_hold_for_their_source_and_configuration(monkeypatch, n, workload):
    """HBM bytes and issued VALU instructions per launch, the second reported
    beside the rate at which the method's lookups are dealt with: one pair for
    each launch configuration in the summary, none for another or for another
    kernel source."""
    sys.path.insert(0, ROOT)
    import bench
    text = open(os.path.join(ROOT, "profiles", "k_stage_q8_%s_pmc.txt" % workload)).read()
    lines = [dict(kv.split("=") for kv in ln.split()[1:]) for ln in re.findall("^traffic:.*$", text, re.M)]
    assert lines
    monkeypatch.setattr(bench, "kernels_source_hash", lambda: lines[0]["kernels_sha256"])
    for v in lines:
        target, wide = int(v["target"]), int(v["wide"])
        nbytes, insts = bench.counted("k_stage", 8, n, target, wide)
        assert nbytes == 1024.0 * (float(v["fetch_kib"]) * float(v["fetch_scale"]) +
                                   float(v["write_kib"]) * float(v["write_scale"]))
        assert insts == float(v["valu_insts"])
        assert bench.counted("k_stage", 8, n, target, 1 - wide) == (None, None)
    assert bench.counted("k_stage", 8, n, 7, wide) == (None, None)
    assert bench.counted("k_diag", 8, n, target, wide) == (None, None)
    monkeypatch.setattr(bench, "kernels_source_hash", lambda: "0" * 16)
    assert bench.counted("k_stage", 8, n, target, wide) == (None, None)
