"""The library's host code over a runtime without a GPU (host_runtime.hip):
plans are really built, in host memory, and launches are recorded instead of
run.  For what the host decides -- tables, routes, launch shapes; outputs stay
as they were."""
import ctypes
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

HERE = os.path.dirname(os.path.abspath(__file__))


class _Launch:
    def __init__(self, rt, i):
        v = (ctypes.c_longlong * 4)()
        self.name = rt.lib.host_runtime_launch(i, v).decode()
        self.grid, self.block, self.lds, self.allowed = list(v)
        self.index = i


class HostRuntime:
    def __init__(self, lib):
        self.lib = lib
        lib.host_runtime_launch.restype = ctypes.c_char_p

    def reset(self):
        self.lib.host_runtime_reset()

    def device(self, d):
        self.lib.host_runtime_device(d)

    def elapsed(self, ms):
        a = (ctypes.c_float * len(ms))(*ms)
        self.lib.host_runtime_elapsed(a, len(ms))

    def launches(self, part=""):
        all_ = [_Launch(self, i) for i in range(self.lib.host_runtime_launches())]
        return [l for l in all_ if part in l.name]

    def team(self, launch):
        """The team tables of a k_pcg_team launch (views of the plan's memory)."""
        names = ("B", "n", "slices", "max_n", "cap_off", "cap", "colcut", "dcol", "dense_cut", "dense_list", "dense_slot",
                 "dense_slots", "used", "uses", "At_loc", "At_rowptr", "At_col", "sliceA", "rowsA", "m")
        v = (ctypes.c_longlong * len(names))()
        self.lib.host_runtime_team(launch.index, v)
        t = dict(zip(names, v))
        BV = t["B"] * t["slices"]
        for k, n, dt in (("colcut", BV + 1, np.int64), ("dcol", t["n"], np.int32), ("dense_cut", BV + 1, np.int64),
                         ("dense_slot", t["n"], np.int32), ("used", 2 * BV, np.int64), ("At_rowptr", t["n"] + 1, np.int64),
                         ("sliceA", 3 * (BV + 1), np.int64), ("rowsA", t["m"], np.int32)):
            t[k] = array(t[k], n, dt) if t[k] else None
        if t["dense_cut"] is not None:
            t["dense_list"] = array(t["dense_list"], int(t["dense_cut"][-1]), np.int32)
        nnz = int(t["At_rowptr"][-1])
        t["At_loc"], t["At_col"] = array(t["At_loc"], nnz, np.uint16), array(t["At_col"], nnz, np.int32)
        return t


def build(out_dir, src_dir=None):
    """Compiles the host side of every source and links it with the runtime."""
    from paper_2606_13825_amd import build as b
    csrc = src_dir or b.CSRC
    flags = ["-O1", "-std=c++17", "-fPIC", f"--offload-arch={b.ARCH}", "--cuda-host-only", "-I", b.INCLUDE, "-I", csrc]

    def one(src):
        obj = os.path.join(out_dir, os.path.basename(src).replace(".hip", ".o"))
        subprocess.run([b.hipcc()] + flags + ["-c", src, "-o", obj], check=True, capture_output=True)
        return obj
    with ThreadPoolExecutor(8) as ex:
        objs = list(ex.map(one, [os.path.join(csrc, s) for s in b.SOURCES] + [os.path.join(HERE, "host_runtime.hip")]))
    # each object refers to its device code, which is not there
    syms = subprocess.run(["nm", "-u"] + objs, check=True, capture_output=True, text=True).stdout
    fat = sorted({w for w in syms.split() if w.startswith("__hip_fatbin")})
    lib = os.path.join(out_dir, "libcosmo_host.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-o", lib] + objs +
                   [f"-Wl,--defsym={s}=0" for s in fat] + ["-lpthread"], check=True, capture_output=True)
    return lib


def load(tmp, monkeypatch, lib=None):
    """The binding over the host runtime, on CPU tensors."""
    from paper_2606_13825_amd import _lib, binding
    cdll = ctypes.CDLL(lib or build(str(tmp)))
    _lib._sig(cdll)
    monkeypatch.setattr(_lib, "_lib", cdll)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda device=None: None)
    monkeypatch.setattr(binding, "_stream", lambda device: ctypes.c_void_p(0))
    return HostRuntime(cdll)


def array(ptr, n, dtype):
    """n elements at an address of the runtime's memory."""
    return np.ctypeslib.as_array((np.ctypeslib.as_ctypes_type(dtype) * n).from_address(ptr))
