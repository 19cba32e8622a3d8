"""Builds host-only headers of the library into a small shared object, so that a CPU test can call what they decide."""
import ctypes
import subprocess
import tempfile
from pathlib import Path

CSRC = Path(__file__).resolve().parent.parent / "paper_2605_11186_amd" / "csrc"


def build(source: str) -> ctypes.CDLL:
    """source: C++ that includes the headers and exports extern "C" functions."""
    with tempfile.TemporaryDirectory() as tmp:
        src, lib = Path(tmp) / "shim.cpp", Path(tmp) / "shim.so"
        src.write_text(source)
        subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(lib)], check=True)
        return ctypes.CDLL(str(lib))
