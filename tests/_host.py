"""Compiles a snippet of C++ that includes the library's host-computable headers
and loads it (no GPU and no HIP needed)."""
import ctypes
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_04302_amd", "csrc")


def have_compiler():
    return shutil.which("g++") is not None


def compile_host(source, folder):
    src, lib = os.path.join(str(folder), "snippet.cpp"), os.path.join(str(folder), "snippet.so")
    with open(src, "w") as f:
        f.write(source)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib],
                   check=True, timeout=120)
    return ctypes.CDLL(lib)
