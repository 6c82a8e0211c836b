"""Planning makes no HIP call: containers, plans and batches can be created before a program
forks or chooses its device. The HIP functions that the library imports are replaced, in a
process of its own, by ones that count their calls and fail."""

import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PLANNING = """
import ctypes, sys
counter = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import paper_2306_12141_amd as rc
from paper_2306_12141_amd import _lib
from paper_2306_12141_amd.batch import Batch, default_tuning
calls = lambda: ctypes.c_int.in_dll(counter, "hip_calls").value
s = (np.arange(200_000) * 7919 % 251).astype(np.uint8)
blobs = [rc.encode(s[:n], lanes=w, quant_bits=b, splits=k) for n, w, b, k in
         ((200_000, 32, 11, 64), (150_001, 64, 12, 40), (90_000, 32, 14, 9), (64, 32, 8, 1))]
for b in blobs:
    rc.Plan(b)
    rc.Plan(rc.Blob.from_bytes(b.to_bytes()), packed_target=0)
for tuning in (None, default_tuning(), _lib.Tuning(8, 8, 1, 0, 2)):
    batch = Batch(blobs, tuning)
    ranges = [batch.output_range(i) for i in range(batch.count)]
    assert batch.workspace_bytes > 0 and batch.tuning.waves in (8, 16)
    t = _lib.Tuning(8, 4, 1, 0, 0)
    _lib.check(_lib.recoil_batch_set_tuning(batch._h, ctypes.byref(t), None, None), "set_tuning")
    assert batch.tuning.waves == 8
assert calls() == 0, calls()
assert batch.items > 0        # the items depend on the device: these are for a whole chip
assert calls() > 0            # (the replacements are in use)
print("ok")
"""


def test_planning_makes_no_hip_call(tmp_path):
    lib = os.path.join(ROOT, "paper_2306_12141_amd", "librecoil.so")
    names = {line.split()[-1].split("@")[0] for line in
             subprocess.run(["nm", "-D", "--undefined-only", lib], check=True, capture_output=True, text=True).stdout.splitlines()}
    hip = sorted(n for n in names if n.startswith("hip") and n not in ("hipGetErrorString", "hipGetErrorName"))
    assert "hipGetDevice" in hip
    src = tmp_path / "count.c"
    src.write_text("int hip_calls = 0;\n" + "".join(f"int {n}(void) {{ ++hip_calls; return 100; }}\n" for n in hip))
    so = tmp_path / "count.so"
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", PLANNING, str(so)], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
