"""Builds libprism_gemm.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB_PATH = os.path.join(_HERE, "libprism_gemm.so")
# the same library with a workgroup barrier after every LDS phase of the main loops, and a full wait
# where the lanes of one wave pass data through LDS (race check: its results must equal the normal
# build's bit for bit)
PARANOID_LIB_PATH = os.path.join(_HERE, "libprism_gemm_paranoid.so")
# the usual call from Python, without ctypes (a module of this package, for the interpreter that builds it)
CALL_PATH = os.path.join(_HERE, "_call" + sysconfig.get_config_var("EXT_SUFFIX"))
_UNITS = ["kernels.hip", "skinny.hip", "dealt.hip", "host_api.hip", "scan.hip", "probe.hip"]
_PARANOID_UNITS = ["kernels.hip", "skinny.hip", "dealt.hip"]  # the units that have such phases
_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    # keep the compiler from forming packed fp32 vector ops out of scalar float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def _sources():
    out = [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if not f.endswith(".o")]
    out.append(os.path.join(os.path.dirname(_HERE), "include", "prism_gemm.h"))
    out.append(os.path.join(os.path.dirname(_HERE), "include", "prism_scan.h"))
    return out


def is_stale() -> bool:
    built = (LIB_PATH, PARANOID_LIB_PATH, CALL_PATH)
    if not all(os.path.exists(p) for p in built):
        return True
    t = min(os.path.getmtime(p) for p in built)
    return any(os.path.getmtime(s) > t for s in _sources())


def build(force: bool = False, verbose: bool = False) -> str:
    """Compile every translation unit and link the shared library.  Returns its path."""
    if not force and not is_stale():
        return LIB_PATH
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    def obj(unit, paranoid=False):
        return os.path.join(CSRC, unit.replace(".hip", "_paranoid.o" if paranoid else ".o"))

    def compile_one(job):
        unit, paranoid = job
        extra = ["-DPRISM_PARANOID_BARRIERS"] if paranoid else []
        cmd = [hipcc, *_FLAGS, *extra, "-c", os.path.join(CSRC, unit), "-o", obj(unit, paranoid)]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {unit}:\n{r.stdout}\n{r.stderr}")
        if "warning:" in r.stderr:
            print(r.stderr, file=sys.stderr, flush=True)

    def compile_call(_):
        cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-Wall",
               "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "call.cpp"), "-o", CALL_PATH]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"call.cpp: {r.stdout}\n{r.stderr}")

    jobs = [(u, False) for u in _UNITS] + [(u, True) for u in _PARANOID_UNITS]
    with ThreadPoolExecutor(max_workers=len(jobs) + 1) as ex:
        call = ex.submit(compile_call, None)
        list(ex.map(compile_one, jobs))
        call.result()
    for lib, paranoid in ((LIB_PATH, False), (PARANOID_LIB_PATH, True)):
        these = [obj(u, paranoid and u in _PARANOID_UNITS) for u in _UNITS]
        cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *these, "-o", lib]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    return LIB_PATH


if __name__ == "__main__":
    print(build(force=True, verbose=True))
