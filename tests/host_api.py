"""The library's host code with stand-ins for the HIP runtime and the kernels'
launches (tests/host_stubs.cpp), compiled for the CPU."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
E_HIP = -3


def build(folder):
    """A fresh copy of the library in `folder`, loaded."""
    lib = os.path.join(str(folder), "host_api.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread",
                    "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"), "-o", lib,
                    os.path.join(ROOT, "paper_2205_15311_amd", "csrc", "jatam_api.cpp"),
                    os.path.join(ROOT, "tests", "host_stubs.cpp")],
                   check=True, capture_output=True, text=True)
    return ctypes.CDLL(lib)


class Host:
    """The loaded library's entry points, and the stand-ins' variables as attributes."""
    TYPES = {"solo_ms": ctypes.c_double, "pipeline_ms": ctypes.c_double,
             "now_ms": ctypes.c_double, "last_n": ctypes.c_longlong}

    def __init__(self, lib):
        object.__setattr__(self, "lib", lib)

    def var(self, name):
        return self.TYPES.get(name, ctypes.c_int).in_dll(self.lib, name)

    def __getattr__(self, name):
        return self.var(name).value

    def __setattr__(self, name, value):
        self.var(name).value = value

    def count(self, call):
        """What a call launches: (one launches, pipelines, shape histograms, graph replays)."""
        names = ("solo_launches", "pipeline_launches", "shape_hists", "graph_launches")
        before = [self.var(n).value for n in names]
        assert call() == 0
        return tuple(self.var(n).value - b for n, b in zip(names, before))
