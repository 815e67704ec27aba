"""Little device memory: where the column reduction of a cloud has just room,
the sweep that is tried before it, and gives up, does not take that room. In
processes of their own, so that the scratch memory starts empty."""

import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRIPT = """
import hashlib, sys
import torch
import paper_1908_02518_amd as r
import workloads
from tests.method_of import method_of
leave, flags = int(sys.argv[1]), int(sys.argv[2])
x = torch.from_numpy(workloads.integer_lattice(440, 3, 440, side=9)).cuda()
small = torch.from_numpy(workloads.sphere(300, 1)).cuda()
r.barcode_device(small, max_dim=0)
out = torch.empty(1 << 22, device="cuda")  # room for the results in torch's own memory
del out
if leave:
    hog = torch.empty(torch.cuda.mem_get_info()[0] - leave, dtype=torch.uint8, device="cuda")
r.set_sweep(flags)
before = torch.cuda.mem_get_info()[0]
(bars, _), s, c = method_of(lambda: r.barcode_device(x, max_dim=2, cap=1 << 14))
used = before - torch.cuda.mem_get_info()[0]
h = hashlib.sha1(b"".join(t.cpu().numpy().tobytes() for b in bars for t in b)).hexdigest()
print("RESULT", used, h, "/".join(sorted(s)) or "-", "/".join(sorted(c)) or "-")
"""


def run(leave, flags):
    p = subprocess.run([sys.executable, "-c", SCRIPT, str(leave), str(flags)], cwd=ROOT, capture_output=True, text=True,
                       timeout=90, env={**os.environ, "PYTHONPATH": ROOT})
    assert p.returncode == 0, p.stdout[-500:] + p.stderr[-1500:]
    used, h, sweeps, columns = next(ln for ln in p.stdout.splitlines() if ln.startswith("RESULT")).split()[1:]
    return int(used), h, sweeps, columns


def test_columns_find_room_after_a_sweep_that_gave_up():
    print("[case] memory: columns alone", flush=True)
    need, want, sweeps, columns = run(0, 0)
    assert sweeps == "-" and "reduce_d2" in columns
    print(f"[case] memory: both methods, room for {need >> 20} MiB and 32 more", flush=True)
    _, got, _, columns = run(need + (32 << 20), 3)
    assert "reduce_d2" in columns
    assert got == want


AFTER_A_BATCH = """
import hashlib
import torch
import paper_1908_02518_amd as r
import workloads
from tests.method_of import method_of
x = torch.from_numpy(workloads.so3(4000, 3)).cuda()
pts = torch.from_numpy(workloads.sphere(512, 2)).cuda()
r.barcode_device(pts[:300], max_dim=0)
before = torch.cuda.mem_get_info()[0]
r.barcode_batched(pts, torch.arange(0, 513, 8, device="cuda"), 2048, max_dim=1)
held = before - torch.cuda.mem_get_info()[0]
out = torch.empty(1 << 25, device="cuda")
del out
hog = torch.empty(torch.cuda.mem_get_info()[0] - (300 << 20), dtype=torch.uint8, device="cuda")
results = []
for _ in range(2):
    (bars, _), s, c = method_of(lambda: r.barcode_device(x, max_dim=2, threshold=1.2, cap=1 << 19))
    results.append(hashlib.sha1(b"".join(t.cpu().numpy().tobytes() for b in bars for t in b)).hexdigest())
    del bars
del hog
torch.cuda.empty_cache()
r.set_sweep(0)
bars, _ = r.barcode_device(x, max_dim=2, threshold=1.2, cap=1 << 19)
results.append(hashlib.sha1(b"".join(t.cpu().numpy().tobytes() for b in bars for t in b)).hexdigest())
print("RESULT", held, "/".join(sorted(s)) or "-", len(set(results)))
"""


def test_a_sweep_finds_the_room_of_another():
    """The scratch memory of a batch is given back where a cloud's sweep needs
    some, before the columns (44 GB here) are thought of."""
    print("[case] memory: a sweep after a large batch", flush=True)
    p = subprocess.run([sys.executable, "-c", AFTER_A_BATCH], cwd=ROOT, capture_output=True, text=True, timeout=90,
                       env={**os.environ, "PYTHONPATH": ROOT})
    assert p.returncode == 0, p.stdout[-500:] + p.stderr[-1500:]
    held, sweeps, distinct = next(ln for ln in p.stdout.splitlines() if ln.startswith("RESULT")).split()[1:]
    assert int(held) > 4 << 30
    assert sweeps == "sweep_d1/sweep_d2" and distinct == "1"
