"""The instrumented build (libpsk_trace.so): bench.py --cu-trace runs in a process of its own (a process loads one
of the two libraries), on a small matrix; every workgroup must have left a record and the busy times must be sane."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_cu_trace_report_on_a_small_matrix():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--workload", "expskew", "--skew-rows", "4096",
                        "--skew-nnz", "400000", "--cu-trace"], capture_output=True, text=True, timeout=300, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    rec = json.loads([l for l in r.stdout.splitlines() if l.startswith("{")][-1])
    names = [s["schedule"] for s in rec["schedules"]]
    assert any("position cut" in n for n in names) and any("wave per row" in n for n in names)
    for s in rec["schedules"]:
        assert s["workgroups"] > 0 and 1 <= s["compute_units"] <= 256
        assert s["max_over_mean"] >= 1.0 and s["cu_busy_us"]["max"] <= s["span_us"] + 0.02
    cut = next(s for s in rec["schedules"] if "position cut" in s["schedule"])
    assert cut["workgroups"] == -(-400000 // 2048) or abs(cut["workgroups"] - 400000 // 2048) <= 2


def test_plain_build_has_no_trace():
    import paper_2001_00532_amd as psk

    assert psk.lib().psk_cu_trace_set(None, 0) == 5          # PSK_ERR_UNSUPPORTED in libpsk.so


def test_small_product_leaves_records():
    """A product that is taken in blocks of whole rows: one record per block (2000 rows of 10: 25 blocks of 80 rows)."""
    code = """
import torch
import paper_2001_00532_amd as psk
psk.use_instrumented_library()
pos = torch.arange(2001, dtype=torch.int32, device="cuda") * 10
crd = torch.zeros(20000, dtype=torch.int32, device="cuda")
one = torch.ones(20000, device="cuda")
y = torch.empty(2000, device="cuda")
records = torch.zeros(3 * (1024 + 64), dtype=torch.int64, device="cuda")
psk.psk_cu_trace_set(records)
psk.psk_spmv_csr(2000, 1, 20000, pos, crd, one, one, y)
torch.cuda.synchronize()
psk.psk_cu_trace_set(None)
r = records.view(-1, 3)[1024:]
assert int((r[:, 1] > 0).sum()) == 25 and bool((r[:25, 1] >= r[:25, 0]).all()) and bool((y == 10).all())
"""
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
