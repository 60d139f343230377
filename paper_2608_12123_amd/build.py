"""Build the HIP library ``librc_cohort.so`` (gfx950) in-tree with hipcc, and
the binding's native caller ``_rc_call`` where the interpreter's headers and a
C compiler are there."""
from __future__ import annotations

import os
import shutil
import subprocess
import sysconfig
import warnings
from typing import Optional

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRC = os.path.join(PKG, "csrc", "rc_cohort.hip")
SRC_HOST = [os.path.join(PKG, "csrc", "rc_host.cpp"),   # descriptor checks and launch plan
            os.path.join(PKG, "csrc", "rc_pack.cpp")]   # cohort shares and online compactor
SRC_CALL = os.path.join(PKG, "csrc", "rc_call.c")          # CPython caller of the chain entry points
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "librc_cohort.so")
# named for the interpreter it is built for, so that another one does not load it
CALL_LIB = os.path.join(PKG, "_rc_call" + sysconfig.get_config_var("EXT_SUFFIX"))
ARCH = "gfx950"

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", "--offload-arch=" + ARCH,
    # packed FP32 instructions are kept out of all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; the HIP library cannot be built")


def build(verbose: bool = False) -> str:
    """Compile ``csrc/rc_cohort.hip``, ``csrc/rc_host.cpp`` and
    ``csrc/rc_pack.cpp`` into ``librc_cohort.so`` (always)."""
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc()] + HIPCC_FLAGS + ["-I", INCLUDE, "-o", tmp, SRC] + SRC_HOST
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    os.replace(tmp, LIB)
    build_call(verbose)
    return LIB


def build_call(verbose: bool = False) -> Optional[str]:
    """Compile ``csrc/rc_call.c`` into the extension module ``_rc_call`` (host
    C, always).  Where that is not possible (no C compiler, no Python headers)
    this warns and returns None: the binding then marshals with ctypes."""
    for old in (CALL_LIB, os.path.join(PKG, "_rc_call.so")):  # never one of other sources
        if os.path.exists(old):
            os.remove(old)
    cc = next((c for c in (shutil.which("cc"), shutil.which("gcc"), hipcc()) if c), None)
    tmp = CALL_LIB + ".tmp%d" % os.getpid()
    cmd = [cc, "-O2", "-std=c11", "-fPIC", "-shared", "-Wall", "-I", sysconfig.get_paths()["include"],
           "-I", INCLUDE, "-o", tmp, SRC_CALL]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
        failed = "" if res.returncode == 0 else "exit status %d\n" % res.returncode + res.stdout + res.stderr
    except OSError as e:
        failed = str(e)
    if failed:
        warnings.warn("the native caller _rc_call is not built; calls go through ctypes:\n" + failed)
        return None
    os.replace(tmp, CALL_LIB)
    return CALL_LIB


if __name__ == "__main__":
    print(build(verbose=True))
