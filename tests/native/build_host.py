"""Builds the library's host code against a stand-in for the HIP runtime
(host_runtime.cpp), for tests of schedules, routes and launches without a device.

The shared library lands in tests/native/_build/libmudiff_host.so; ``Host`` loads it
and keeps what the library launches."""
from __future__ import annotations

import concurrent.futures as cf
import ctypes
import fcntl
import os
import subprocess
import sys
import weakref

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
sys.path.insert(0, ROOT)

from paper_1409_8186_amd import _lib as L  # noqa: E402
from paper_1409_8186_amd import build as libbuild  # noqa: E402

OUT = os.path.join(HERE, "_build", "host")
LIB = os.path.join(HERE, "_build", "libmudiff_host.so")


def _run(cmd: list) -> str:
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{' '.join(cmd)}:\n{r.stderr}")
    return r.stdout


def build() -> str:
    os.makedirs(OUT, exist_ok=True)
    with open(os.path.join(OUT, "lock"), "w") as lock:  # one test process at a time
        fcntl.flock(lock, fcntl.LOCK_EX)
        return _build()


def _build() -> str:
    flags = [libbuild.HIPCC, f"--offload-arch={libbuild.ARCH}", "--offload-host-only", "-O1", "-std=c++17", "-fPIC",
             "-Wno-unused-result"]

    def compile_one(src: str) -> str:
        obj = os.path.join(OUT, os.path.basename(src).rsplit(".", 1)[0] + ".o")
        _run([*flags, "-c", src, "-o", obj])
        return obj

    srcs = libbuild.sources() + [os.path.join(HERE, "host_runtime.cpp")]
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(compile_one, srcs))
    # the embedded device code, which is not built here
    names = {w for o in objs for w in _run(["nm", "-u", o]).split() if w.startswith("__hip_fatbin_")}
    stub = os.path.join(OUT, "fatbin.c")
    with open(stub, "w") as f:
        f.write("".join(f"char {n}[8];\n" for n in sorted(names)))
    # -Bsymbolic: the stand-in also where the process holds the HIP runtime
    _run(["g++", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-o", LIB + ".tmp", *objs, "-x", "c", stub])
    os.replace(LIB + ".tmp", LIB)
    return LIB


class Memory:
    """256-byte aligned memory that stands for the device's (not touched)."""

    def __init__(self, n: int):
        self.data = np.empty(n + 256, np.uint8)
        self.base = self.data.ctypes.data + -self.data.ctypes.data % 256
        self.n = n


class Host:
    """The library on the stand-in: ``launches`` holds (kernel, blocks, threads, LDS bytes,
    stream) of every launch, and ``hooks`` maps a part of a kernel's name to a function
    called with (read(index, ctype), blocks) at its launch.  Copies to the device are refused
    outside the memory that ``array`` handed out."""

    def __init__(self):
        self.lib = ctypes.CDLL(build())
        for name, (res, args) in L.SIGNATURES.items():
            fn = getattr(self.lib, name)
            fn.restype, fn.argtypes = res, args
        self.launches, self.hooks, self.arrays = [], {}, weakref.WeakSet()
        self.keep = []
        launch = ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.c_uint, ctypes.c_uint, ctypes.c_uint, ctypes.c_uint,
                                  ctypes.c_size_t, ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p))
        self._launch = launch(self._on_launch)
        self.lib.host_on_launch(self._launch)
        self._copy = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t)(self._on_copy)
        self.lib.host_on_copy(self._copy)
        self._clock = ctypes.CFUNCTYPE(ctypes.c_float)

    def _on_launch(self, name, gx, gy, gz, threads, lds, stream, args):
        name = name.decode()
        self.launches.append((name, (gx, gy, gz), threads, lds, stream))
        for part, fn in self.hooks.items():
            if part in name:
                fn(lambda k, t: ctypes.cast(args[k], ctypes.POINTER(t))[0], (gx, gy, gz))

    def _on_copy(self, dst, n):
        return 0 if any(a.base <= dst and dst + n <= a.base + a.n for a in self.arrays) else 1

    def clock(self, f) -> None:
        """f() is what the next timed event pair says, in ms."""
        self._elapsed = self._clock(f)
        self.lib.host_on_elapsed(self._elapsed)

    def check(self, status: int) -> None:
        if status:
            raise L.MudiffError(status, self.lib.mudiff_last_error().decode())

    def array(self, n_bytes: int) -> Memory:
        m = Memory(int(n_bytes))
        self.arrays.add(m)
        return m

    def tables(self, instances, circulant: bool = False):
        """Handle of instances (centers, radii, n_modes, k)."""
        off = np.cumsum([0] + [len(i[1]) for i in instances]).astype(np.int64)
        c = np.ascontiguousarray(np.concatenate([np.asarray(i[0], float).reshape(-1, 2) for i in instances]))
        a = np.concatenate([np.asarray(i[1], float) for i in instances])
        n = np.concatenate([np.asarray(i[2], np.int32) for i in instances])
        k = np.array([float(i[3]) for i in instances])
        flags = L.TABLES_CIRCULANT if circulant else 0
        size = self.lib.mudiff_tables_workspace_size(len(instances), off.ctypes.data, n.ctypes.data, flags)
        assert size > 0
        ws = self.array(size)
        h = ctypes.c_void_p()
        self.check(self.lib.mudiff_tables(len(instances), off.ctypes.data, c.ctypes.data, a.ctypes.data, n.ctypes.data,
                                          k.ctypes.data, ws.base, size, flags, None, ctypes.byref(h)))
        self.keep = [ws]  # as long as the handle: one at a time
        return h
