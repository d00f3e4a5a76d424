"""Fields and populations read back without pinned host memory, or without host
threads, are the same bit for bit.  Needs an MI355X."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = """
import ctypes, sys
deny = ctypes.CDLL(%r, ctypes.RTLD_GLOBAL)
sys.path[:0] = [%r, %r]
import numpy as np
from gpu_helpers import B, smooth_fields
b = B()
for lattice, prec, sizes in (("d2q9", "fp64", [(40, 30)]), ("d2q9", "fp32", [(1201, 1003)]),
                             ("d2q9", "fp16dev", [(9, 7), (700, 301), (64, 64), (650, 811)]), ("d1q3", "fp64", [(900001, 1)])):
    q = 9 if lattice == "d2q9" else 3
    params = [b.make_params(lattice, "srt", "periodic", prec, nx, ny, 0.7) for nx, ny in sizes]
    fields = [smooth_fields(nx, ny, seed=k) for k, (nx, ny) in enumerate(sizes)]
    rho, ux, uy = (np.concatenate([f[i].reshape(-1) for f in fields]) for i in range(3))
    got = []
    for pinned, threads in ((1, 0), (0, 1), (0, 0)):
        c = b.lbm_init(params[0], rho, ux, uy) if len(sizes) == 1 else b.lbm_init_batch(params, rho, ux, uy)
        b.lbm_step(c, 5)
        n = deny.denied()
        deny.deny(pinned, threads)
        got.append((*b.lbm_moments(c), b.lbm_get_populations(c, q)))
        deny.deny(0, 0)
        print(lattice, sizes, pinned, threads, deny.denied() - n, flush=True)
        assert (deny.denied() > n) == bool(pinned or (threads and sum(x * y for x, y in sizes) > 500000))
        b.lbm_free(c)
    for g in got[:2]:
        assert all(np.array_equal(x, y) for x, y in zip(g, got[2]))
print("same")
"""


def test_without_pinned_memory_or_threads(tmp_path):
    lib = str(tmp_path / "libdenier.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "hip_denier.cpp"), "-o", lib, "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD % (lib, HERE, os.path.dirname(HERE))], capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and r.stdout.rstrip().endswith("same"), r.stdout + r.stderr
