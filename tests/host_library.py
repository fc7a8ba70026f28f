"""libscocg.so on the host, without a device: a program that runs it on the runtime of host_runtime.cpp.

    run(program, tmp_path)

The program finds `C` (the ctypes declarations), `lib` (the library), `fake` (the runtime's switches and
records), `np`, and the helpers below.
"""

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, importlib.util, os, sys
import numpy as np
fake = ctypes.CDLL({shim!r}, ctypes.RTLD_GLOBAL)
fake.fake_live.restype = ctypes.c_size_t
fake.fake_name.restype = ctypes.c_char_p
fake.fake_threads_x.restype = ctypes.c_uint64
fake.fake_set_limit.argtypes = [ctypes.c_size_t]
spec = importlib.util.spec_from_file_location('scocg_capi', {capi!r})
C = importlib.util.module_from_spec(spec)
spec.loader.exec_module(C)
lib = C.load()
SEED_STOPPED = 3  # every status read back: the block loop ends at its first look
OUT = ctypes.c_void_p(1 << 42)  # stands for a device output


def launched(part):
    return sum(part in fake.fake_name(i).decode() for i in range(fake.fake_launches()))


def band(n, width):
    # (row_ptr, col, val) of a symmetric band with `width` entries a row, wrapped around
    h = (width - 1) // 2
    col = np.sort((np.arange(n)[:, None] + np.arange(-h, h + 1)) % n, axis=1).astype(np.int64)
    return np.arange(n + 1, dtype=np.int64) * (2 * h + 1), col.ravel(), np.ones(col.size)


def upload(rp, col, val):
    H = ctypes.c_void_p()
    rc = lib.csr_upload(len(rp) - 1, len(col), rp.ctypes.data, col.ctypes.data, val.ctypes.data, 0, None, ctypes.byref(H))
    return rc, H


def hubbard(L, n_up, n_dn):
    H = ctypes.c_void_p()
    assert lib.hubbard_upload(L, n_up, n_dn, 1.0, 4.0, 1.0, None, ctypes.byref(H)) == C.OK
    return H


def greens(H, K, M=2, entry='greens_diag', **opts):
    # a call whose right-hand sides all stop in the first block
    fake.fake_set_word(SEED_STOPPED)
    o = C.Opts()
    lib.scocg_default_opts(ctypes.byref(o))
    for k, v in opts.items():
        setattr(o, k, v)
    z = np.linspace(-1, 1, M) + 0.5j
    idx = np.zeros(K, dtype=np.int64)
    args = [H, M, z.ctypes.data, K, idx.ctypes.data, ctypes.byref(o), OUT, None]
    return getattr(lib, entry)(*args, *([None] if entry == 'greens_diag' else []), None)


def krylov_vec(H, nu=2):
    fake.fake_set_word(1)  # (the start vector's norm is not zero)
    z = np.array([0.5j])
    return lib.krylov_greens_vec(H, 1, z.ctypes.data, OUT, nu, OUT, None, None, None)
"""


def run(program, tmp_path):
    shim = os.path.join(os.path.dirname(str(tmp_path)), "host_runtime.so")  # once per session
    if not os.path.exists(shim):
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                               "-I/opt/rocm/include", os.path.join(HERE, "host_runtime.cpp"), "-o", shim])
    capi = os.path.join(ROOT, "paper_0802_0748_amd", "_capi.py")
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(shim=shim, capi=capi) + program], cwd=ROOT,
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-4000:])
    return r.stdout
