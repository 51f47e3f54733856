"""Compiles a test's .hip file for the host alone, against the library's own headers and with its flags, and loads it."""
import ctypes
import importlib.util
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def load(name, out_dir):
    spec = importlib.util.spec_from_file_location("agal_build", os.path.join(ROOT, "paper_2502_16310_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    lib = os.path.join(str(out_dir), f"lib{name}.so")
    cmd = [build.HIPCC, *build.CXXFLAGS, "--offload-host-only", "-w", "-shared", "-Wl,-Bsymbolic",
           os.path.join(ROOT, "tests", f"{name}.hip"), "-o", lib]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(lib)
