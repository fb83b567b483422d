"""Builds the C-ABI library ``libkvev.so`` from ``csrc/*.hip`` with hipcc for gfx950.

Run as ``python -m paper_2509_21354_amd.build`` (add ``--force`` to recompile
everything).  Objects go to ``_build/`` next to this file; the shared library
and the extension module ``_native`` (marshalling, built with g++; optional:
without it calls go through ctypes) stay in-tree next to the sources so that
they travel with the checkout.
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
OBJ_DIR = os.path.join(_HERE, "_build")
LIB_PATH = os.path.join(_HERE, "libkvev.so")
# CPython module: marshalling of calls into the library (its name says which Python it is for)
NATIVE_PATH = os.path.join(_HERE, "_native" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # packed fp32 VALU forms stay off (device-code feature; the host pass ignores it)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _headers_mtime():
    hs = glob.glob(os.path.join(CSRC, "*.hpp")) + glob.glob(os.path.join(_HERE, "..", "include", "*.h"))
    return max(os.path.getmtime(h) for h in hs)


def _compile(src: str, obj: str) -> str:
    cmd = [HIPCC, *FLAGS, *os.environ.get("KVEV_EXTRA_FLAGS", "").split(), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {os.path.basename(src)}:\n{r.stdout}\n{r.stderr}")
    noise = "is not a recognized feature for this target"
    return "\n".join(line for line in r.stderr.splitlines() if noise not in line)


def _build_native(force: bool, hdr: float) -> None:
    src = os.path.join(CSRC, "native_call.cpp")
    if not force and os.path.exists(NATIVE_PATH) and os.path.getmtime(NATIVE_PATH) >= max(os.path.getmtime(src), hdr):
        return
    cmd = [CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", sysconfig.get_paths()["include"], src, "-o", NATIVE_PATH]
    try:
        subprocess.run(cmd, check=True, capture_output=True, text=True)
    except (OSError, subprocess.CalledProcessError) as e:
        if os.path.exists(NATIVE_PATH):          # (an old one may not fit the library)
            os.remove(NATIVE_PATH)
        print(f"the marshalling extension is not built, calls will go through ctypes: {e}\n{getattr(e, 'stderr', '')}", file=sys.stderr)


def build(force: bool = False, verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    hdr = _headers_mtime()
    jobs, objs = [], []
    for src in _sources():
        obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        stale = force or not os.path.exists(obj) or os.path.getmtime(obj) < max(os.path.getmtime(src), hdr)
        if stale:
            jobs.append((src, obj))
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, max(1, len(jobs)))) as ex:
        for warn in ex.map(lambda j: _compile(*j), jobs):
            if warn.strip() and verbose:
                print(warn, file=sys.stderr)
    _build_native(force, hdr)
    if jobs or not os.path.exists(LIB_PATH):
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs])
    return LIB_PATH


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
