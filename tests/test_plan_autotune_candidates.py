"""The shapes that the autotuner of one plan tries: for few runs also the throughput kernel's, which
a cap on resident workgroups asks for. The HIP functions that the library imports are replaced, in
a process of its own, by ones that do nothing; the replaced clock makes one candidate after the
other the fastest."""

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
fastest, timed = (ctypes.c_int.in_dll(shim, n) for n in ("fastest", "timed"))
s = (np.arange(3_000_000) * 7919 % 251).astype(np.uint8)
fake = ctypes.c_void_p(256)
for units in (2048, 5000, 9000):
    seen, k, total = set(), 0, 1
    while k < total:
        # (A length of its own each: results are cached by the stream's shape.)
        plan = rc.Plan(rc.encode(s[:units * 96 + k], lanes=32, quant_bits=11, splits=units))
        fastest.value, timed.value = k, 0
        best, ms = _lib.Tuning(), ctypes.c_float()
        _lib.check(_lib.recoil_plan_autotune(plan._h, fake, fake, fake, None, 1, ctypes.byref(best), ctypes.byref(ms)), "autotune")
        assert ms.value == 0.5
        seen.add((best.waves, best.chunk_groups, best.blocks_per_cu, best.units_per_run))
        total = timed.value
        k += 1
    assert len(seen) == total
    few = lambda r: -(-units // max(r, 1)) <= 2048
    assert seen == {(w, K, cap, r) for w in (1, 8, 16) for K in (4, 8) for r in (0, 1, 2, 4)
                    for cap in (0, 32 // w) if cap == 0 or (w < 16 and few(r))}, (units, sorted(seen))
print("ok")
"""


def test_autotuner_tries_both_kernels_for_few_runs(tmp_path):
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
