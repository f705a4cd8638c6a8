"""Runs a piece of Python in a process of its own in which libllr.so calls
tests/csrc/hip_recorder.cpp instead of the HIP runtime (no GPU, no kernels), and
hands it the recorded calls."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = '''
import ctypes as C, json, sys
import numpy as np
from paper_1509_08391_amd import llr
rec = C.CDLL(None)
for f, r in (("rec_count", C.c_long), ("rec_news", C.c_long), ("rec_new_max", C.c_size_t), ("rec_op", C.c_char_p),
             ("rec_name", C.c_char_p), ("rec_stream", C.c_void_p), ("rec_bytes", C.c_size_t)):
    getattr(rec, f).restype = r
for f in ("rec_op", "rec_name", "rec_stream", "rec_bytes"):
    getattr(rec, f).argtypes = [C.c_long]
rec.rec_fail.argtypes = [C.c_char_p, C.c_long]
L = llr.lib()

def calls():
    """(kind, kernel, stream, bytes) of every call since the last reset"""
    return [(rec.rec_op(i).decode(), rec.rec_name(i).decode(), rec.rec_stream(i) or 0, rec.rec_bytes(i))
            for i in range(rec.rec_count())]

def dptr(a):
    return a.ctypes.data_as(C.POINTER(C.c_double))

def context(prec=llr.FP64, lats=(), order=llr.SWEEP_GROUPED, stream=0x77, **params):
    """A context with its state bound (of zeros) and its tiles set"""
    h = C.c_void_p()
    assert L.llr_create(C.byref(h), 0, C.c_void_p(stream), prec) == 0
    p = dict(n_th=2, n_a=4, n_rm=100, seed=5, replica_exchange=0, overlap=1.0, recompute_every=10, eps=1e-4,
             approach_cap=100)
    p.update(params)
    assert L.llr_set_params(h, C.byref(llr.Params(*p.values()))) == 0
    assert L.llr_set_sweep_order(h, order) == 0
    for size, n in lats:
        v6 = 6.0 * size ** 4
        e = 0.5 * v6 + 0.2 * v6 / n * np.arange(n)
        assert L.llr_add_lattice(h, size, n, dptr(e), 0.2 * v6 / n, None) == 0
    if lats:
        nb = C.c_size_t()
        assert L.llr_state_bytes(h, C.byref(nb)) == 0
        raw = np.zeros(nb.value + 256, dtype=np.uint8)
        at = (raw.ctypes.data + 255) // 256 * 256
        assert L.llr_bind_state(h, C.c_void_p(at), nb.value) == 0
        assert L.llr_set_tiles(h, 2, 2) == 0
        keep.append(raw)
    return h

keep = []
'''


def run(tmp_path, body):
    """body sets `result` (JSON values), which is returned."""
    so = str(tmp_path / "hip_recorder.so")
    b = subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "csrc", "hip_recorder.cpp"),
                        "-o", so], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([sys.executable, "-c", PRELUDE + body + "\nprint('RESULT' + json.dumps(result))\n"], cwd=ROOT,
                       env=dict(os.environ, LD_PRELOAD=so), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
    return json.loads(r.stdout.rsplit("RESULT", 1)[1])
