"""Generated kernels on the CPU (wave_emu.h): compiles the source of the last plan for the host and runs it on buffers that
end at an inaccessible page."""
import ctypes
import os
import re
import subprocess

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = next((p for p in ("/opt/rocm/llvm/bin/clang++", "/opt/rocm/bin/amdclang++") if os.path.exists(p)), "clang++")
MAX_SIDES = 8


class Args(ctypes.Structure):
    """fuse_kargs (csrc/fuse_args.h)"""
    _fields_ = [("x", ctypes.c_void_p), ("colidx", ctypes.c_void_p), ("rowptr", ctypes.c_void_p),
                ("side", ctypes.c_void_p * MAX_SIDES), ("side_ld", ctypes.c_longlong * MAX_SIDES),
                ("side_scalar", ctypes.c_double * MAX_SIDES), ("u", ctypes.c_void_p), ("v", ctypes.c_void_p),
                ("ldu", ctypes.c_longlong), ("ldv", ctypes.c_longlong),
                ("m", ctypes.c_longlong), ("n", ctypes.c_longlong), ("ld", ctypes.c_longlong), ("nnz", ctypes.c_longlong),
                ("out", ctypes.c_void_p), ("partials", ctypes.c_void_p), ("ticket", ctypes.c_void_p),
                ("rank", ctypes.c_int), ("npanels", ctypes.c_int), ("panel_ptr", ctypes.c_void_p),
                ("panel_w", ctypes.c_int), ("block_rows", ctypes.c_int), ("row_limit", ctypes.c_longlong),
                ("side_ci", ctypes.c_void_p * MAX_SIDES),
                ("side_rp", ctypes.c_void_p * MAX_SIDES)]


class Kernels:
    """The kernels `names` of a generated source, compiled into `folder`; defines override those of the source."""

    def __init__(self, source, folder, names, defines=None):
        fields = re.search(r"typedef struct \{(.*?)\} fuse_kargs;", source, flags=re.S).group(1)
        fields = re.sub(r"/\*.*?\*/", "", fields, flags=re.S)
        declared = [n for n in re.findall(r"\*?(\w+)(?:\[FUSE_MAX_SIDES\])?\s*[,;]", fields)]
        assert declared == [f[0] for f in Args._fields_], declared
        source = re.sub(r"asm volatile\([^;]*\);", "", source)
        source = re.sub(r"__attribute__\(\(amdgpu_waves_per_eu\([^)]*\)\)\)", "", source)
        for k, v in (defines or {}).items():
            source, n = re.subn(r"^#define %s .*$" % k, "#define %s %s" % (k, v), source, flags=re.M)
            assert n == 1, k
        self.source = source
        wrap = "".join('extern "C" void emu_%s(const void *a) { %s(*(const fuse_kargs *)a); }\n' % (n, n) for n in names)
        path = os.path.join(str(folder), "kernel_%s.cpp" % names[0])
        with open(path, "w") as f:
            f.write('#include "wave_emu.h"\n' + source + "\n" + wrap)
        out = path[:-4] + ".so"
        subprocess.run([CLANG, "-std=c++17", "-O1", "-ffp-contract=off", "-fno-strict-aliasing", "-fPIC", "-shared", "-w",
                        "-U_FORTIFY_SOURCE", "-I", HERE, path, "-o", out, "-lm"], check=True)
        self.lib = ctypes.CDLL(out)
        self.lib.emu_alloc.restype = ctypes.c_void_p
        self.lib.emu_alloc.argtypes = [ctypes.c_size_t]
        self.lib.emu_run.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint, ctypes.c_uint, ctypes.c_int]
        self.lib.emu_error.restype = ctypes.c_char_p

    def define(self, name):
        return int(re.search(r"^#define %s (\d+)" % name, self.source, flags=re.M).group(1))

    def buffer(self, shape, dtype=np.float64):
        """An array whose last byte is followed by the inaccessible page (rounded up to 16 bytes), all zeros."""
        dtype = np.dtype(dtype)
        count = int(np.prod(shape))
        p = self.lib.emu_alloc(max(count * dtype.itemsize, 1))
        assert p, "no address space"
        raw = (ctypes.c_char * (count * dtype.itemsize)).from_address(p)
        a = np.frombuffer(raw, dtype=dtype).reshape(shape)
        return a

    def copy(self, a, dtype=None):
        a = np.asarray(a, dtype=dtype)
        b = self.buffer(a.shape, a.dtype)
        b[...] = a
        return b

    def run(self, name, args, blocks, threads, last_first=False):
        rc = self.lib.emu_run(ctypes.cast(getattr(self.lib, "emu_" + name), ctypes.c_void_p), ctypes.byref(args), blocks, threads,
                              int(last_first))
        assert rc == 0, self.lib.emu_error().decode()
