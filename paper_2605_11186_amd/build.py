"""Build step: compiles the HIP sources for gfx950 into libcats.so (in-tree)."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
ROOT = PKG.parent
LIB = PKG / "libcats.so"
SOURCES = ["fused_swiglu.hip", "fused_qkv.hip", "gemm.hip", "gemv.hip", "rowops.hip", "attention.hip", "accept.hip", "loss.hip", "api.hip"]


def _run(cmd: list[str]) -> str:
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        print(res.stdout)
        print(err)
        raise RuntimeError("hipcc failed")
    return res.stdout + err


def build_library(verbose: bool = False) -> Path:
    """One object per source, compiled side by side, then linked."""
    base = ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC"]
    flags = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             f"-I{ROOT / 'include'}", f"-I{PKG / 'csrc'}"]
    with tempfile.TemporaryDirectory() as tmp:
        objs = [str(Path(tmp) / f"{s}.o") for s in SOURCES]
        cmds = [base + flags + ["-c", str(PKG / "csrc" / s), "-o", o] for s, o in zip(SOURCES, objs)]
        with ThreadPoolExecutor(min(len(cmds), os.cpu_count() or 1)) as pool:
            logs = list(pool.map(_run, cmds))
        logs.append(_run(base + ["-shared", *objs, "-o", str(LIB)]))
    if verbose:
        print("\n".join(logs))
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
