"""Runs a function of a test on the library over ``host_runtime.c``, in a
process of its own (the stand-in has to be loaded before the library)."""

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def build(out_dir) -> str:
    so = os.path.join(str(out_dir), "libhostruntime.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    os.path.join(HERE, "host_runtime.c"), "-o", so], check=True)
    return so


def run(so: str, module: str, name: str, *args):
    """``module.name(rt, *args)``, rt being the stand-in's handle."""
    code = ("import ctypes as C, importlib, sys\n"
            f"rt = C.CDLL({so!r}, mode=C.RTLD_GLOBAL)\n"
            "rt.rt_limit.argtypes = [C.c_size_t]\n"
            "rt.rt_used.restype = rt.rt_peak.restype = C.c_size_t\n"
            "rt.rt_launches.restype = rt.rt_instantiated.restype = C.c_longlong\n"
            f"sys.path.insert(0, {ROOT!r})\n"
            f"importlib.import_module({module!r}).{name}(rt, *{args!r})\n")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
