"""libadiwave.so on the recording HIP runtime (hip_recorder.c), without a GPU.

run(body) executes `body` in a process of its own, with `lib` (the C ABI), `_lib`, `ct`
(ctypes), `rec` (the recorder) and the helpers below, and returns what it assigns to `out`
(plain values)."""
import atexit
import functools
import json
import os
import shutil
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "hip_recorder.c")

PRELUDE = '''
import ctypes as ct, json, sys
sys.path.insert(0, {root!r})
rec = ct.CDLL({so!r}, mode=ct.RTLD_GLOBAL)      # before the library: its HIP calls bind here
rec.rec_log.restype = ct.c_char_p
rec.rec_set_rmax.argtypes = [ct.c_double]
from paper_2006_10142_amd import _lib
lib = _lib.load()
A, B, C, D = 1 << 44, 2 << 44, 3 << 44, 4 << 44   # "device" addresses nothing reads

def wave(nx, ny, rmax, f64=False):
    rec.rec_set_rmax(rmax)
    h = ct.c_void_p()
    _lib.check(lib.adi_wave_create(ct.byref(h), nx, ny, 0.1, 0.1, None, 1.0, int(f64), None))
    return h

def names():
    """kernels (and memcpys) queued since the last call"""
    got = [l.split()[0] for l in rec.rec_log().decode().splitlines()]
    rec.rec_clear()
    return got

def short(ks):
    """symbol names without scope and arguments: k_fusedr, k_xsweep ..."""
    import re
    return [(re.findall(r"\\d(k_[a-z0-9_]+)", k) or [k])[0] for k in ks]

def step(w, n=1):
    names()
    a, b = ct.c_void_p(A), ct.c_void_p(B)
    _lib.check(lib.adi_wave_step(w, ct.byref(a), ct.byref(b), None, None, n))
    return names()

def info(w):
    i = _lib.AdiWaveInfo()
    _lib.check(lib.adi_wave_get_info(w, ct.byref(i)))
    return {{f: getattr(i, f) for f, _ in i._fields_}}

def tune(w, **kw):
    return lib.adi_wave_set_tuning(w, ct.byref(_lib.AdiTuning(**kw)))
'''


@functools.lru_cache(maxsize=None)
def build() -> str:
    folder = tempfile.mkdtemp(prefix="adiwave_recorder_")
    atexit.register(shutil.rmtree, folder, ignore_errors=True)
    so = os.path.join(folder, "recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, SRC], check=True)
    return so


def run(body: str):
    code = PRELUDE.format(root=ROOT, so=build()) + body + "\nprint('OUT' + json.dumps(out))\n"
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert p.returncode == 0, p.stdout[-2000:] + p.stderr[-4000:]
    return json.loads([l for l in p.stdout.splitlines() if l.startswith("OUT")][-1][3:])
