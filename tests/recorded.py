"""Runs a piece of Python against liblbm.so on top of the recording runtime of
hip_recorder.cpp, in a process of its own (CPU only; nothing is executed on a
device).  The piece sees the binding as `B`, numpy as `np`, the recorder as
`rec`, and `kernels()`, which returns and clears the launches since the last
call as (short kernel name, grid x, grid y, block x)."""
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, re, sys, types
rec = ctypes.CDLL(%(recorder)r, ctypes.RTLD_GLOBAL)
rec.rec_name.restype = ctypes.c_char_p
rec.rec_name.argtypes = [ctypes.c_long]
rec.rec_count.restype = rec.rec_blocks.restype = rec.rec_events.restype = ctypes.c_long
rec.rec_grid.argtypes = rec.rec_block.argtypes = [ctypes.c_long, ctypes.c_int]
rec.rec_grid.restype = rec.rec_block.restype = ctypes.c_uint
rec.rec_refuse.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_int]
# the binding asks torch only for the current stream and for pointers
torch = types.ModuleType("torch")
torch.cuda = types.SimpleNamespace(is_available=lambda: False)
sys.modules["torch"] = torch
sys.path.insert(0, %(root)r)
import numpy as np
from paper_1801_03863_amd import binding as B

def kernels():
    out = []
    for i in range(rec.rec_count()):
        m = re.match(r"_ZN3lbm\\d+(k_[a-z0-9_]+?)(I|E)", rec.rec_name(i).decode())
        out.append((m.group(1) if m else "?", rec.rec_grid(i, 0), rec.rec_grid(i, 1), rec.rec_block(i, 0)))
    rec.rec_clear()
    return out

def single(lattice, coll, bc, prec, nx, ny):
    p = B.make_params(lattice, coll, bc, prec, nx, ny, 0.6, 0.0, 0.05 if bc == "cavity" else 0.0, 1.0)
    z = np.zeros(nx * ny)  # never read: uploads do nothing
    return B.lbm_init(p, z, z, z, stream=0)

def batch(lattice, coll, bc, prec, sizes):
    p = [B.make_params(lattice, coll, bc, prec, nx, ny, 0.6, 0.0, 0.0, 1.0) for nx, ny in sizes]
    z = np.zeros(sum(nx * ny for nx, ny in sizes))
    return B.lbm_init_batch(p, z, z, z, stream=0)

def shapes(ctx, word):
    return [v for v in range(B.lbm_variant_count(ctx)) if word in B.lbm_variant_name(ctx, v)]
"""


def build_recorder(folder):
    out = os.path.join(str(folder), "librecorder.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-Wno-unused-result", os.path.join(HERE, "hip_recorder.cpp"), "-o", out, "-ldl"], check=True)
    return out


def run(recorder, body, timeout=100):
    """Run `body` and return what it prints; fails if it raises."""
    code = PRELUDE % {"recorder": recorder, "root": ROOT} + re.sub(r"(?m)^    ", "", body)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=timeout, cwd=ROOT)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
