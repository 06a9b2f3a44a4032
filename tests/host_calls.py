"""Runs a script against libtsgemm in a process whose HIP runtime only records
(tests/hip_record.cpp).  The script finds: `lib` (the library's binding),
`launches()` (what was launched since the last call), `rec` (the recorder),
`on(fn)` (calls fn once, at the next launch or capture query)."""
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PRELUDE = '''
import ctypes, threading
from paper_1905_03136_amd import _lib as lib
lib.lib()
rec = ctypes.CDLL(None)
rec.rec_buffer.restype = ctypes.c_uint64
rec.rec_buffer.argtypes = [ctypes.c_uint64]
class Record(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", ctypes.c_uint32), ("block", ctypes.c_uint32), ("shmem", ctypes.c_uint64),
                ("stream", ctypes.c_uint64), ("args", ctypes.c_uint64 * 12)]
    def is_(self, kernel):
        return kernel.encode() in self.name
def launches():
    out = []
    for i in range(rec.rec_count()):
        r = Record()
        rec.rec_get(i, ctypes.byref(r))
        out.append(r)
    rec.rec_clear()
    return out
_hook_type = ctypes.CFUNCTYPE(None, ctypes.c_char_p)
def on(where, fn):
    def hook(w):
        if w == where.encode():
            rec.rec_hook(ctypes.cast(None, _hook_type))
            fn()
    on.keep = _hook_type(hook)
    rec.rec_hook(on.keep)
A, B, C, S = 1 << 46, 1 << 45, 1 << 43, 64   # addresses, a stream
'''


def run(tmp_path, script):
    stub = os.path.join(str(tmp_path), "libhiprecord.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "hip_record.cpp"), "-o", stub], check=True)
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(script)], cwd=ROOT, text=True, timeout=300,
                       env=dict(os.environ, LD_PRELOAD=(stub + " " + os.environ.get("LD_PRELOAD", "")).strip(),
                                PYTHONPATH=ROOT), stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT)
    assert r.returncode == 0, r.stdout[-4000:]
    return r.stdout
