"""libpf over a HIP runtime of the tests' own (hip_stub.cpp): what its host code
asks a device for, on a machine without one.  Run in a process of its own, as a
process holds one HIP runtime only: `run(code)` executes the text with `lib`,
`stub` and the helpers below in scope."""
from __future__ import annotations

import ctypes as C
import functools
import os
import subprocess
import sys
import textwrap

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
OUT = os.path.join(ROOT, "_build")
SO = os.path.join(OUT, "libhipstub.so")
LIB_PATH = os.environ.get("PF_LIBPF") or os.path.join(ROOT, "paper_1811_02512_amd", "libpf.so")


@functools.lru_cache(maxsize=None)
def build():
    os.makedirs(OUT, exist_ok=True)
    tmp = f"{SO}.{os.getpid()}.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-Wl,-soname,libamdhip64.so.7",
                    os.path.join(HERE, "hip_stub.cpp"), "-o", tmp], check=True)
    os.replace(tmp, SO)


def run(code):
    """Runs `code` against the stub; its asserts are the test's."""
    build()
    head = "from tests.stub_runtime import *\nlib, stub = load()\n"
    r = subprocess.run([sys.executable, "-c", head + textwrap.dedent(code)], cwd=ROOT, text=True,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=300)
    assert r.returncode == 0, r.stdout
    return r.stdout


# ---- in the child process --------------------------------------------------
def load():
    global lib, stub
    stub = C.CDLL(SO, mode=C.RTLD_GLOBAL)
    lib = C.CDLL(LIB_PATH)
    lib.pf_last_error.restype = C.c_char_p
    return lib, stub


class Info(C.Structure):  # pf_info
    _fields_ = ([(k, C.c_int32) for k in ("n", "m", "nn", "slack")] +
                [(k, C.c_int64) for k in ("nnz_y", "nnz_l", "n_upd")] +
                [(k, C.c_int32) for k in ("nlevels", "max_level_width")] +
                [(k, C.c_int64) for k in ("vals_doubles", "ws_doubles")] +
                [("dev_bytes", C.c_size_t)] +
                [(k, C.c_int32) for k in ("tail_levels", "tail_nodes", "tail_lds_bytes",
                                          "threads", "tail_clique", "ws_interleave")] +
                [(k, C.c_int64) for k in ("lu_offset", "fd_mat_doubles", "fd_ws_doubles")] +
                [(k, C.c_int32) for k in ("spread", "sub_levels")])


class Sym:
    """A grid's symbolic, in host memory standing for the device's."""

    def __init__(self, g, threads=0, budget=65536):
        i32 = lambda a: np.ascontiguousarray(a, np.int32)
        f, t = i32(g.f), i32(g.t)
        self.h = C.c_void_p()
        assert lib.pf_analyze(g.n, f.size, vp(f), vp(t), 0, 0, C.byref(self.h)) == 0
        assert lib.pf_symbolic_set_launch(self.h, threads, C.c_int64(budget), 1) == 0
        assert self.upload() == 0

    @property
    def info(self):
        i = Info()
        assert lib.pf_symbolic_info(self.h, C.byref(i)) == 0
        return i

    def upload(self, bytes=None):
        n = self.info.dev_bytes if bytes is None else bytes
        self.buf = np.zeros(n + 256, np.uint8)
        at = (self.buf.ctypes.data + 255) & ~255
        return lib.pf_symbolic_upload(self.h, C.c_void_p(at), C.c_size_t(n), None)


def vp(a):
    return a.ctypes.data_as(C.c_void_p)


def latest():
    """(kernel, workgroups, threads, dynamic LDS) of this thread's latest launch."""
    name, out = C.create_string_buffer(128), (C.c_longlong * 3)()
    stub.stub_latest(name, 128, out)
    return (name.value.decode(), *out)


PTR = C.c_void_p(1 << 20)  # an argument that is checked and passed on, not read
I64, D = C.c_int64, C.c_double


def mismatch(s, B=1):
    n = s.info.n
    return lib.pf_mismatch(s.h, B, PTR, I64(0), PTR, I64(0), PTR, PTR, I64(0), PTR, PTR, I64(n),
                           PTR, I64(2 * n), PTR, None, None)


def fdpf(s, B=1):
    i = s.info
    return lib.pf_fdpf(s.h, B, PTR, I64(0), PTR, I64(0), PTR, PTR, I64(0), PTR, PTR, I64(i.n), PTR,
                       I64(i.fd_mat_doubles), D(1e-8), 40, PTR, I64(i.fd_ws_doubles), None, None,
                       None, None)
