"""Build libflashblock.so (hand-written HIP for gfx950) and libfbcalib.so (the benchmark's calibration
kernels: read and MFMA ceilings, a plain copy) in-tree with hipcc, and _fbcall (the Python binding's native marshalling, an extension module
for this interpreter) with gcc.  The libraries need no compiler but hipcc: without gcc or Python's headers the binding goes through ctypes.

    python -m paper_2602_05305_amd.build [--force]

The libraries are written next to this file so that they travel with the source tree; nothing is
installed.  Objects go to paper_2602_05305_amd/_build/ (ignored by git).
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libflashblock.so")
CALIB_LIB = os.path.join(HERE, "libfbcalib.so")
# host code only: the binding's native marshalling.  Named for the interpreter it is compiled for: another one does not load it.
CALL_LIB = os.path.join(HERE, "_fbcall" + sysconfig.get_config_var("EXT_SUFFIX"))
CALIB_SOURCES = ["fb_calib.hip"]
SOURCES = ["fb_api.hip", "fb_attn_f32.hip", "fb_attn_bf16.hip", "fb_stream_bf16.hip", "fb_aux.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # the direct-to-LDS loads set M0 from inline assembly and say so in the clobber list
         "-Wno-inline-asm",
         # keep the compiler from forming packed fp32 VALU ops
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l).strip()
    if err:
        sys.stderr.write(err + "\n")
    return obj


def _newest_source() -> float:
    newest = max(os.path.getmtime(os.path.join(CSRC, f)) for f in os.listdir(CSRC))
    return max(newest, os.path.getmtime(os.path.join(HERE, "..", "include", "flashblock.h")))


def _fresh(*files: str) -> bool:
    return all(os.path.exists(f) and os.path.getmtime(f) >= _newest_source() for f in files)


def _build_call() -> None:
    """The binding's native marshalling; where it cannot be built, none is left from before and the libraries work without it."""
    for old in (CALL_LIB, os.path.join(os.path.dirname(CALL_LIB), "_fbcall.so")):
        if os.path.exists(old):
            os.remove(old)
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "fb_call.c"), "-o", CALL_LIB]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
        failed = f"{r.stdout}\n{r.stderr}" if r.returncode != 0 else ""
    except OSError as e:
        failed = str(e)
    if failed:
        sys.stderr.write(f"fb_call.c is not built, calls go through ctypes: {failed}\n")


def build(force: bool = True) -> str:
    """Compile every HIP source for gfx950 and link the shared libraries.  Returns the path of libflashblock.so."""
    os.makedirs(OBJ, exist_ok=True)
    if force or not _fresh(LIB, CALIB_LIB):
        with ThreadPoolExecutor(max_workers=6) as ex:
            objs = list(ex.map(_compile, SOURCES + CALIB_SOURCES))
        for lib, lobjs in ((LIB, objs[:len(SOURCES)]), (CALIB_LIB, objs[len(SOURCES):])):
            cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *lobjs]
            r = subprocess.run(cmd, capture_output=True, text=True)
            if r.returncode != 0:
                raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    if force or not _fresh(CALL_LIB):
        _build_call()
    return LIB


if __name__ == "__main__":
    print(build(force=True))
