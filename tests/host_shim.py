"""Host-side rules of the library (plain C++ headers under csrc/), compiled with the host compiler for tests without a GPU."""
import ctypes
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_08666_amd", "csrc")


def load(folder, source):
    """The shared library of a C++ source that includes such headers."""
    cpp, so = os.path.join(str(folder), "shim.cpp"), os.path.join(str(folder), "shim.so")
    with open(cpp, "w") as f:
        f.write(source)
    subprocess.check_call([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, cpp, "-o", so])
    return ctypes.CDLL(so)
