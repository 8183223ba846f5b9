"""libadmm.so on a HIP runtime without a device (fake_hip.c): what the host code
allocates and launches, without a GPU. Runs in a process of its own, because the
library binds its runtime once: `run(code)` executes code there with `fake` (the
runtime's counters), `admm` and `init` defined and returns what it prints."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
sys.path.insert(0, {root!r})
fake = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
for f in ("fake_used", "fake_largest", "fake_lds_most", "fake_shape_hash"):
    getattr(fake, f).restype = ctypes.c_size_t
fake.fake_event_ms.argtypes = [ctypes.c_double, ctypes.c_double]
fake.fake_reset.argtypes = [ctypes.c_size_t]
from paper_2010_06697_amd import admm
UNLIMITED = (1 << 64) - 1
keep = []


def init(shapes, precision, **params):
    '''(status, context) of admm_init with host fields, mu = 1, lambda = 4.'''
    rves = []
    for n3, n2, n1 in shapes:
        r, V, s = admm.Rve(), n1 * n2 * n3, 8 if precision == admm.FP64 else 4
        r.n[0], r.n[1], r.n[2] = n1, n2, n3
        for name, size in (("phase", V), ("u", 24 * V), ("u_prev", 24 * V), ("F", 9 * V * s),
                           ("Lambda", 9 * V * s)):
            keep.append(ctypes.create_string_buffer(size))
            setattr(r, name, ctypes.addressof(keep[-1]))
        for k in range(9):
            r.Fbar[k] = float(k % 4 == 0)
        rves.append(r)
    p = admm.default_params("fp64" if precision == admm.FP64 else "fp32", **params)
    ctx = ctypes.c_void_p()
    rc = admm.lib().admm_init(ctypes.byref(ctx), (admm.Rve * len(rves))(*rves), len(rves),
                              (admm.Material * 1)(admm.material(mu=1.0, lam=4.0)), 1,
                              ctypes.byref(p), precision, None, 0, None)
    return rc, ctx
"""


def run(code, tmp_path):
    lib = os.path.join(str(tmp_path), "libfakehip.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", os.path.join(HERE, "fake_hip.c"), "-o", lib],
                   check=True)
    p = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, lib=lib) + code],
                       capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr
    return p.stdout
