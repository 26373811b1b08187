"""The library's host code on a machine without a GPU: libfstat.so loaded on a stand-in for
the HIP runtime (hip_stub.cpp) in a process of its own.  `run(body)` runs Python statements
there with `H`, this module's Host: the library's C ABI, the kernels launched so far and a
place to let calls fail or to act for a kernel."""
from __future__ import annotations

import ctypes
import os
import re
import shutil
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SO = "libamdhip64.so.7"
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def build(folder) -> str:
    from paper_1410_3677_amd import fstat as F
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(F.LIB_PATH) or not os.path.exists(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs g++, the HIP headers and the built library")
    out = os.path.join(str(folder), SO)
    subprocess.run([gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-w",
                    f"-Wl,-soname,{SO}", "-I", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", "hip_stub.cpp"), "-o", out], check=True)
    return out


def run(stub: str, body: str) -> str:
    """The statements' standard output; an assertion that fails there fails here."""
    code = f"from tests.hip_stub import Host\nH = Host({stub!r})\n" + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


class Host:
    def __init__(self, stub):
        # loaded first, it serves the library's dependency of the same name
        self.stub = ctypes.CDLL(stub, mode=ctypes.RTLD_GLOBAL)
        from paper_1410_3677_amd import fstat as F
        self.F, self.lib = F, F.load()
        self.launches = []        # (kernel, grid x, grid y, grid z, workgroup x)
        self.on = {}              # runtime call or kernel name -> function of its arguments; returns an error code
        kind = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_char_p, ctypes.c_char_p, ctypes.POINTER(ctypes.c_longlong),
                                ctypes.POINTER(ctypes.c_void_p))

        def hook(what, detail, dims, args):
            what, name = what.decode(), re.sub(r"^void |^fstat::", "", detail.decode())
            name = re.sub(r"^fstat::", "", name)
            if what == "launch":
                self.launches.append((name.split("(")[0], *dims[0:4]))
                what = re.split(r"[<(]", name)[0]
            f = self.on.get(what)
            return int(f(args) or 0) if f else 0
        self._hook = kind(hook)
        self.stub.stub_set_hook(self._hook)
        self._mem = ctypes.create_string_buffer(1 << 20)
        self.ptr = (ctypes.addressof(self._mem) + 255) & ~255   # "device" memory that is never looked into

    def names(self):
        return [v[0] for v in self.launches]

    def plan(self, lengths, **opts):
        F = self.F
        segs = (F.fstat_segment * len(lengths))(*[F.fstat_segment(n, 2.0, 100.0, 1.0, self.ptr, self.ptr, 0.8, 3.0, 0.0)
                                                  for n in lengths])
        o = F.fstat_options()
        self.lib.fstat_options_default(ctypes.byref(o))
        o.candidate_capacity = 1 << 14
        for k, v in opts.items():
            setattr(o, k, v)
        h = ctypes.c_void_p()
        r = self.lib.fstat_plan(segs, len(lengths), ctypes.byref(o), ctypes.byref(h))
        assert r == F.OK, (r, self.lib.fstat_last_error(None))
        return h

    def search(self, plan, nsky, nfdot, segment=0):
        return self.lib.fstat_search_batch(plan, segment, self.ptr, self.ptr, nsky, self.ptr, nfdot, None)

    def spectrum(self, plan, nsky, nfdot, static=False):
        f = self.lib.fstat_twoF_spectrum_static if static else self.lib.fstat_twoF_spectrum
        return f(plan, 0, self.ptr, self.ptr, nsky, self.ptr, nfdot, self.ptr, None)

    def workspace(self, plan):
        v = ctypes.c_size_t()
        assert self.lib.fstat_plan_workspace_size(plan, ctypes.byref(v)) == self.F.OK
        return v.value
