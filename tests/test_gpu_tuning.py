"""DA_SPMM_TUNE is read once: what it overrides, seen from a process of its own."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import json, os, sys, tempfile, torch
from torch.profiler import ProfilerActivity, profile
from paper_2202_08556_amd import binding as da
def launches(call):
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    with tempfile.TemporaryDirectory() as d:
        prof.export_chrome_trace(os.path.join(d, "t.json"))
        events = json.load(open(os.path.join(d, "t.json")))["traceEvents"]
    return [(e["name"], e["args"].get("grid")) for e in events if e.get("cat") == "kernel"]
def matrix(lens, k):
    rowptr = torch.zeros(lens.numel() + 1, dtype=torch.int32)
    rowptr[1:] = lens.cumsum(0)
    at = torch.arange(int(rowptr[-1])) - torch.repeat_interleave(rowptr[:-1].long(), lens)
    return rowptr.cuda(), (at % k).to(torch.int32).cuda(), torch.ones(int(rowptr[-1]), device="cuda")
out = {}
m, k, N = 1000, 10007, 128                       # two column tiles, which go to XCDs of their own otherwise
A = matrix(torch.full((m,), 5), k)
B, C = torch.ones((k, N), device="cuda"), torch.empty((m, N), device="cuda")
out["tiles"] = launches(lambda: da.da_spmm(m, k, N, *A, B, C, da.DA_RB_RM_PR))
m, k, N = 1000, 20011, 8                         # rows that have a kernel of their own otherwise
lens = torch.full((m,), 3)
lens[::20] = 15000
A = matrix(lens, k)
B, C = torch.ones((k, N), device="cuda"), torch.empty((m, N), device="cuda")
da.da_spmm_prepare(m, k, A[1].numel(), A[0], A[1])
out["heavy"] = launches(lambda: da.da_spmm(m, k, N, *A, B, C, da.DA_EB_RM_SR))
print(json.dumps(out))
"""


def launched(**env):
    run = subprocess.run([sys.executable, "-c", PROGRAM], cwd=ROOT, env={**os.environ, **env}, capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stderr[-2000:]
    return json.loads(run.stdout.strip().splitlines()[-1])


@pytest.mark.parametrize("tuned", [False, True])
def test_overrides_win(tuned):
    got = launched(**({"DA_SPMM_TUNE": "1", "DA_SPMM_PIN": "0"} if tuned else {}))
    print(got, flush=True)
    grids = [g for name, g in got["tiles"] if "rb_pr_kernel" in name]
    assert len(grids) == 1 and (grids[0] is None or grids[0][1] == (2 if tuned else 1))
    names = " ".join(name for name, _ in got["heavy"])
    assert ("eb_sr_kernel" in names, "heavy_rows_kernel" in names) == (tuned, not tuned)
