"""Occupancy queries that a decode makes on the host, in each range of runs: one for the shape
that is looked at and one for the shape that is launched, at most. The HIP functions that the
library imports are replaced, in a process of its own, by ones that do nothing."""

import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
int queries;
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int %(occupancy)s(int *v) { ++queries; *v = 2; return 0; }
"""

DECODE = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import paper_2306_12141_amd as rc
from paper_2306_12141_amd import _lib
queries = ctypes.c_int.in_dll(shim, "queries")
s = (np.arange(9001 * 64 * 3) * 7919 % 251).astype(np.uint8)
fake = ctypes.c_void_p(256)
for W in (32, 64):
    for M in (1, 256, 1024, 1500, 2049, 4096, 4097, 6000, 8192, 8193, 9000):
        plan = rc.Plan(rc.encode(s[:M * 3 * W], lanes=W, quant_bits=11, splits=M))
        queries.value = 0
        _lib.check(_lib.recoil_decode(plan._h, fake, fake, fake, None), "decode")
        print(W, M, queries.value)
        assert 1 <= queries.value <= 2, (W, M, queries.value)
print("ok")
"""


def test_queries_of_a_decode(tmp_path):
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
    r = subprocess.run([sys.executable, "-c", DECODE, str(so)], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
