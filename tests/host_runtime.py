"""The library's host code on a stand-in HIP runtime (CPU only).

``build`` compiles the library's own sources for the host alone, links them
with tests/hip_stub/stub_hip.cpp in place of the HIP runtime, and returns
the result as a ctypes library with the prototypes of the bindings. Its
kernels are not run; what the host code enqueues, waits for and gives back is
what the tests look at.
"""

import ctypes as C
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2606_23087_amd import build as lib_build
from paper_2606_23087_amd import flowpool as fp

HERE = os.path.dirname(os.path.abspath(__file__))
INCLUDE = os.path.join(lib_build.ROOT, "include")
CSRC = os.path.join(lib_build.HERE, "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
INVALID_VALUE, LAUNCH_FAILURE = 1, 719     # hipErrorInvalidValue, hipErrorLaunchFailure


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return r.stdout


def build(tmp, csrc=CSRC):
    hipcc = lib_build.hipcc()
    if not os.path.exists(hipcc) or not shutil.which("g++") or not shutil.which("nm"):
        pytest.skip("hipcc, g++ or nm not available")
    objs, defs = [], []
    for src in ("pool.hip", "kernels.hip", "schedule.cpp", "allocate.cpp"):
        o = os.path.join(str(tmp), src + ".o")
        hip = ["--cuda-host-only"] if src.endswith(".hip") else []
        _run([hipcc, *hip, "-O1", "-std=c++17", "-fPIC", "-I", INCLUDE, "-I", csrc, "-c", os.path.join(csrc, src), "-o", o])
        # the device code the host objects would carry
        defs += [f"-Wl,--defsym={s}=0" for s in re.findall(r"U (__hip_fatbin\w*)", _run(["nm", o]))]
        objs.append(o)
    stub = os.path.join(str(tmp), "stub.o")
    _run(["g++", "-std=c++17", "-O1", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
          "-c", os.path.join(HERE, "hip_stub", "stub_hip.cpp"), "-o", stub])
    so = os.path.join(str(tmp), "libflowpool_host.so")
    _run(["g++", "-shared", "-Wl,-Bsymbolic", *defs, *objs, stub, "-o", so])
    lib = C.CDLL(so)
    for name, (res, args) in fp._SIGS.items():
        f = getattr(lib, name)
        f.restype, f.argtypes = res, args
    lib.stub_log.restype = C.c_char_p
    lib.stub_migrate_args.restype = C.c_void_p
    return lib


class Pool:
    """A pool of a host build: both tiers, scatter policy, 64-byte rows and pages of 4 rows unless said otherwise."""

    def __init__(self, lib, hbm_pages=64, host_pages=64, hidden=32, page=4, chunk_bytes=0, shuffle=0):
        self.lib, self.page = lib, page
        cfg = fp.fp_pool_config()
        lib.fp_config_init(C.byref(cfg))
        cfg.hidden, cfg.page_tokens, cfg.vocab = hidden, page, 100
        cfg.hbm_pages, cfg.host_pages = hbm_pages, host_pages
        cfg.chunk_bytes, cfg.frame_shuffle_seed = chunk_bytes, shuffle
        cfg.alloc_policy = fp.FP_ALLOC_SCATTER
        self.p = C.c_void_p()
        assert lib.pool_create(C.byref(cfg), C.byref(self.p)) == 0, lib.fp_last_error()

    def write(self, n_text, rows, stream, tiers=(0,)):
        """(status, id); the wished tiers of the pages are `tiers`, repeated."""
        text = (C.c_int32 * max(n_text, 1))()
        one = (C.c_int32 * 1)(0)
        ntok = (C.c_int32 * 1)(rows)
        n = -(-rows // self.page)
        wish = (C.c_uint8 * max(n, 1))(*[tiers[k % len(tiers)] for k in range(n)])
        vis = np.zeros(64, np.int16)
        sid = C.c_uint64()
        st = self.lib.pool_write_sample(self.p, text, n_text, one, ntok, 1, C.c_void_p(_aligned(vis)), wish, stream, sid)
        return st, sid.value

    def ids(self, l):
        return (C.c_uint64 * max(len(l), 1))(*l)

    def plan(self, l, stream):
        n = max(len(l), 1)
        return self.lib.plan_microbatches(self.p, self.ids(l), len(l), 4096, 2, 16, 0, (C.c_int32 * n)(), (C.c_int32 * 2)(),
                                          (C.c_int64 * 2)(), (C.c_int32 * 2)(), (C.c_int64 * n)(), stream)

    def pack(self, l, stream, noalloc=False):
        rows = 1 << 16
        out, table = np.zeros((rows, 32), np.int16), np.zeros((100, 32), np.int16)
        f = self.lib.pack_microbatch_noalloc if noalloc else self.lib.pack_microbatch
        return f(self.p, self.ids(l), len(l), C.c_void_p(_aligned(table)), 100, C.c_void_p(_aligned(out)), rows, None,
                 None, None, None, 3, stream)

    def migrate(self, l, tier, stream):
        return self.lib.pool_migrate(self.p, self.ids(l), len(l), tier, stream, None)

    def stats(self):
        a, b, c = C.c_int64(), C.c_int64(), C.c_int64()
        self.lib.pool_stats(self.p, a, b, c)
        return a.value, b.value, c.value

    def pages(self, i):
        n = C.c_int32()
        buf = (C.c_uint64 * 4096)()
        assert self.lib.pool_sample_pages(self.p, i, buf, 4096, n) == 0
        return list(buf[:n.value])

    def frames(self, i):
        """(tier, address) of each of a sample's pages."""
        out = []
        for g in self.pages(i):
            t, at = C.c_int32(), C.c_uint64()
            assert self.lib.pool_translate(self.p, g, t, at) == 0
            out.append((t.value, at.value))
        return out

    def destroy(self):
        assert self.lib.pool_destroy(self.p) == 0

    def copies(self):
        """(source, destination, bytes) of the asynchronous copies since the last call of log."""
        at = C.POINTER(C.c_ulonglong)()
        n = self.lib.stub_copies(C.byref(at))
        return [(at[3 * k], at[3 * k + 1], at[3 * k + 2]) for k in range(n)]

    def log(self):
        """Lines logged since the last call."""
        l = self.lib.stub_log().decode().split("\n")[:-1]
        self.lib.stub_clear()
        return l


def _aligned(a):
    # nothing reads or writes it: the stand-in runs no kernel
    return (a.ctypes.data + 15) // 16 * 16
