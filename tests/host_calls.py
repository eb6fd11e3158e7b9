"""Runs libsbh's host code without a GPU: the library in a fresh process on the stand-in runtime
(hip_stand_in.cpp), whose log of runtime calls the tests read."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = r'''
import ctypes as C, struct, sys
sys.path.insert(0, ROOT)
H = C.CDLL(STAND_IN, mode=C.RTLD_GLOBAL)
H.stand_in_log.restype = C.c_char_p
H.stand_in_arg.restype = C.c_uint64
H.stand_in_capture.argtypes = [C.c_void_p]
import paper_2506_02219_amd as P
L = P.lib()
GIB = 1 << 30
S1, S2 = C.c_void_p(0x51), C.c_void_p(0x52)   # streams
D = C.c_void_p(1 << 44)                       # some device memory

def log(clear=True):
    """The calls since the last clear: [(name, pointer or event, bytes or threads, stream, device)]."""
    rows = [l.split() for l in H.stand_in_log().decode().splitlines()]
    if clear:
        H.stand_in_clear()
    return [(r[0], int(r[1], 16), int(r[2]), int(r[3], 16), r[4]) for r in rows]

def of(rows, *names):
    return [r for r in rows if r[0] in names]

def levels(*per_level):
    """The sizes that the next builds read back: (nodes, internal nodes) of each level."""
    t = [0] * 44
    for l, (nodes, inner) in enumerate(per_level):
        t[2 * l], t[2 * l + 1] = nodes, inner
    raw = struct.pack("8f44I", 0, 0, 0, 1, 1, 0, 0, 0, *t)
    H.stand_in_info(raw, len(raw))

def build(n=5000, stream=S1, normals=False, **opts):
    o = P.BuildOpts(opts.get("branching", 2), 8, 0, 0, 0)
    h = C.c_void_p()
    st = L.sbh_build(D, D, D if normals else None, n, C.byref(o), stream, C.byref(h))
    assert st == 0, L.sbh_last_error()
    return h

levels((1, 1), (8, 0))
'''


def stand_in(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("stand_in") / "libhip_stand_in.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", lib, os.path.join(HERE, "hip_stand_in.cpp")],
                   check=True)
    return lib


def run(lib, code):
    src = f"ROOT = {ROOT!r}\nSTAND_IN = {lib!r}\n" + PRELUDE + code + "\nprint('host calls ok')\n"
    r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "host calls ok" in r.stdout, (r.returncode, r.stdout[-2000:], r.stderr[-3000:])
