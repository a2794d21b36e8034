"""Build ``libspmd.so`` from the HIP sources in ``csrc/`` for gfx950, and
``_launch.so``, the Python side's launch call, from ``csrc/pylaunch.cpp``.

Every translation unit is compiled with hipcc for gfx950 only, with packed
fp32 instructions disabled, then linked into one shared library next to this
file.  ``python paper_2206_07896_amd/build.py`` rebuilds it.
"""

from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OUT = os.path.join(HERE, "libspmd.so")
LAUNCH_OUT = os.path.join(HERE, "_launch.so")
BUILD_DIR = os.path.join(ROOT, "_build")

ARCH = "gfx950"


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def compile_flags() -> list[str]:
    return [
        f"--offload-arch={ARCH}",
        "-O3",
        "-std=c++17",
        "-fPIC",
        "-Wall",
        "-Wno-unused-function",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", INCLUDE,
        "-I", CSRC,
    ]


def build_launch(verbose: bool = False) -> str:
    """The extension module of the Python launch path (host code only)."""
    tmp = LAUNCH_OUT + f".tmp{os.getpid()}"
    cmd = [os.environ.get("CXX") or shutil.which("g++") or "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-I", sysconfig.get_paths()["include"], "-I", INCLUDE, os.path.join(CSRC, "pylaunch.cpp"), "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"the launch module failed to build:\n{r.stderr}")
    os.replace(tmp, LAUNCH_OUT)
    return LAUNCH_OUT


def build(verbose: bool = False, jobs: int = 8) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    cc = hipcc()

    def one(src: str) -> str:
        obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
        cmd = [cc, "-c", src, "-o", obj] + compile_flags()
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
        return obj

    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        launch = ex.submit(build_launch, verbose)
        objs = list(ex.map(one, srcs))
        launch.result()
    tmp = OUT + f".tmp{os.getpid()}"
    cmd = [cc, "-shared", "-Wl,--no-undefined", f"--offload-arch={ARCH}", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
