"""The shapes that the batch autotuner tries, the default shape among them. The HIP functions
that the library imports are replaced, in a process of its own, by ones that do nothing; the
replaced clock makes one candidate after the other the fastest."""

import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
int fastest, timed;
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int %(occupancy)s(int *v) { *v = 2; return 0; }
int hipEventElapsedTime(float *ms) { *ms = timed++ == fastest ? 0.5f : 1.0f; return 0; }
"""

TUNE = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import paper_2306_12141_amd as rc
from paper_2306_12141_amd import _lib
from paper_2306_12141_amd.batch import Batch, default_tuning
fastest, timed = (ctypes.c_int.in_dll(shim, n) for n in ("fastest", "timed"))
as_tuple = lambda t: tuple(getattr(t, f) for f, _ in t._fields_)
s = (np.arange(60_000) * 7919 % 251).astype(np.uint8)
seen, k, total = set(), 0, 1
while k < total:
    # (A length of its own each: results are cached by the batch's shape.)
    batch = Batch([rc.encode(s[:50_000 + k], lanes=32, quant_bits=11, splits=20)])
    fastest.value, timed.value = k, 0
    best, ms = _lib.Tuning(), ctypes.c_float()
    fake = ctypes.c_void_p(256)
    _lib.check(_lib.recoil_autotune(batch._h, fake, fake, fake, None, 1, ctypes.byref(best), ctypes.byref(ms)), "autotune")
    assert ms.value == 0.5 and as_tuple(batch.tuning) == as_tuple(best)
    seen.add(as_tuple(best))
    total = timed.value
    k += 1
assert len(seen) == total
assert seen == {(w, K, p, 0, r) for w in (8, 16) for K in (4, 8) for p in (1, 2, 4, 8) for r in (0, 1, 2, 4, 8)}, sorted(seen)
assert as_tuple(default_tuning()) in seen
print("ok")
"""


def test_autotuner_tries_the_default_shape(tmp_path):
    lib = os.path.join(ROOT, "paper_2306_12141_amd", "librecoil.so")
    names = {line.split()[-1].split("@")[0] for line in
             subprocess.run(["nm", "-D", "--undefined-only", lib], check=True, capture_output=True, text=True).stdout.splitlines()}
    occupancy = [n for n in names if n.startswith("hip") and "Occupancy" in n]
    assert len(occupancy) == 1
    text = SHIM % {"occupancy": occupancy[0]}
    for n in sorted(names):
        if (n.startswith("hip") or n.endswith("CallConfiguration")) and n != "hipGetErrorString" and f" {n}(" not in text:
            text += f"int {n}(void) {{ return 0; }}\n"
    src, so = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(text)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", TUNE, str(so)], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
