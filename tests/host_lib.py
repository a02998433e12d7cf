"""libhqr's host dispatch without a GPU: the library's sources compiled for the
host only and linked with host_stub.cpp in place of the HIP runtime.  Nothing
runs; what was launched, recorded and waited for is read from a log."""
import concurrent.futures
import ctypes
import os
import re
import subprocess

import numpy as np

from paper_2506_09463_amd import _build

STUB = os.path.join(os.path.dirname(__file__), "host_stub.cpp")
ROCM = os.path.dirname(os.path.dirname(_build.HIPCC))


def _run(cmd):
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-3000:]
    return res.stdout


def build(folder):
    """Path of the host-only library, built in `folder`."""
    inc = ["-I", _build.INCLUDE, "-I", _build.CSRC]
    objs = [os.path.join(folder, os.path.basename(s)[:-4] + ".o") for s in _build.sources()]
    with concurrent.futures.ThreadPoolExecutor(max_workers=4) as ex:
        list(ex.map(lambda so: _run([_build.HIPCC, "--offload-host-only", "-O0", "-std=c++17", "-fPIC"] + inc
                                    + ["-c", so[0], "-o", so[1]]), zip(_build.sources(), objs)))
    # the device images the objects would register
    syms = sorted(set(re.findall(r"U (__hip_fatbin\w*)", _run(["nm", "-u"] + objs))))
    images = os.path.join(folder, "images.c")
    with open(images, "w") as f:
        f.write("".join("char %s[8];\n" % s for s in syms))
    lib = os.path.join(folder, "libhqr_host.so")
    _run(["gcc", "-fPIC", "-c", images, "-o", images[:-2] + ".o"])
    _run(["g++", "-std=c++17", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-c", STUB,
          "-o", os.path.join(folder, "stub.o")])
    _run(["g++", "-shared", "-Wl,-Bsymbolic"] + objs + [images[:-2] + ".o", os.path.join(folder, "stub.o"), "-lpthread",
                                                        "-o", lib])
    return lib


class HostLib:
    def __init__(self, folder):
        self.lib = ctypes.CDLL(build(str(folder)))
        self.lib.host_log.restype = ctypes.c_char_p
        self.lib.host_fail.argtypes = [ctypes.c_char_p, ctypes.c_int]
        self.lib.hqr_tune_set.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 4 + [ctypes.c_int, ctypes.c_int]
        self.lib.hqr_tune_variant_name.restype = ctypes.c_char_p
        self.keep = []

    def log(self, clear=True):
        out = self.lib.host_log().decode().splitlines()
        if clear:
            self.lib.host_clear()
        return out

    def fail(self, name="", nth=0):
        self.lib.host_fail(name.encode(), nth)

    def variant(self, name):
        return [self.lib.hqr_tune_variant_name(i).decode() for i in range(self.lib.hqr_tune_variants())].index(name)

    def batched(self, shapes, factored=None):
        """Status of one batched call on problems of the given (m, n, nrhs)."""
        k = len(shapes)
        i64 = ctypes.c_int64 * k
        ptr = ctypes.c_void_p * k
        m, n, r = ([int(s[j]) for s in shapes] for j in range(3))
        buf = np.zeros(16)
        self.keep = [buf]
        p = ptr(*[buf.ctypes.data] * k)
        info = (ctypes.c_int * k)()
        f = (ctypes.c_int * k)(*(factored or [0] * k))
        return self.lib.qr_lsq_batched_mixed(ctypes.c_int(k), i64(*m), i64(*n), i64(*r), p, i64(*m), p, p, i64(*m), p, f,
                                             info, None, ctypes.c_int64(0), None)

    def factor(self, m, n):
        """Status of qr_factor on an m x n problem, without a workspace."""
        buf = np.zeros(16)
        info = ctypes.c_int()
        p = ctypes.c_void_p(buf.ctypes.data)
        i64 = ctypes.c_int64
        return self.lib.qr_factor(i64(m), i64(n), p, i64(m), p, None, i64(0), ctypes.byref(info), None)

    def apply(self, m, n, nrhs):
        """Status of qr_apply_qt with an m x n factor, without a workspace."""
        buf = np.zeros(16)
        p = ctypes.c_void_p(buf.ctypes.data)
        i64 = ctypes.c_int64
        return self.lib.qr_apply_qt(i64(m), i64(n), i64(nrhs), p, i64(m), p, p, i64(m), None, i64(0), None)

    def lsq(self, m, n, nrhs):
        """Status of qr_lsq_solve on an m x n problem, without a workspace."""
        buf = np.zeros(16)
        info = ctypes.c_int()
        p = ctypes.c_void_p(buf.ctypes.data)
        i64 = ctypes.c_int64
        return self.lib.qr_lsq_solve(i64(m), i64(n), i64(nrhs), p, i64(m), p, p, i64(m), p, None, None, i64(m), None,
                                     i64(0), ctypes.byref(info), None, None)
