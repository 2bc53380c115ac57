"""Builds libabsb.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
_CSRC = os.path.join(_HERE, "csrc")
_INCLUDE = os.path.join(os.path.dirname(_HERE), "include")
_OBJ = os.path.join(_HERE, "_build")
LIB_PATH = os.path.join(_HERE, "libabsb.so")
# the same library for the tests, except that a work-group of the store build hardly waits for the others of its segment:
# the rows of nearly all of them go through memory
NOWAIT_PATH = os.path.join(_HERE, "libabsb_nowait.so")

# -packed-fp32-ops is switched off on purpose (v_pk_*_f32 forms are not trusted on this target);
# the host pass does not know the feature and says so, which is harmless.
_COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           # leading kernel arguments arrive in scalar registers (the dispatcher fetches them ahead of the first wave)
           "-mllvm", "-amdgpu-kernarg-preload-count=14",
           "-Wall", "-Wextra", "-Wno-unused-parameter", f"-I{_INCLUDE}", f"-I{_CSRC}"]
# per-file extras: the files that decide integers keep every binary32 step a single IEEE operation
_SOURCES = {
    "api.hip": [],
    "build.hip": ["-ffp-contract=off"],
    "score.hip": ["-ffp-contract=off"],
    "topk.hip": [],
    "decode.hip": ["-ffp-contract=off"],   # FMAs are written explicitly there
    "fused.hip": ["-ffp-contract=off"],    # holds the estimation stage too
    "own.hip": ["-ffp-contract=off"],      # likewise
    "shared.hip": ["-ffp-contract=off"],   # likewise
    "small.hip": ["-ffp-contract=off"],    # likewise
    "util.hip": [],
}


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


# host-side sanitizers (the device pass is left alone: -Xarch_host applies each flag to the host compile only)
_HOST_SANITIZE = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host",
                  "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer", "-g"]


def _compile(name: str, extra, obj_name: str = "") -> str:
    obj = os.path.join(_OBJ, obj_name or name.replace(".hip", ".o"))
    cmd = [_hipcc(), *_COMMON, *extra, "-c", os.path.join(_CSRC, name), "-o", obj]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {name}:\n{out}")
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj


def build_sanitized(jobs: int = 8) -> str:
    """libabsb_san.so: the same sources with AddressSanitizer + UndefinedBehaviorSanitizer on the HOST
    code (argument validation, planning, workspace carving, Eq. (2)), for CPU-only test runs under the
    clang sanitizer runtime.  Returns its path."""
    global _OBJ, LIB_PATH
    keep = (_OBJ, LIB_PATH)
    _OBJ, LIB_PATH = os.path.join(_HERE, "_build_san"), os.path.join(_HERE, "libabsb_san.so")
    try:
        os.makedirs(_OBJ, exist_ok=True)
        with ThreadPoolExecutor(max_workers=jobs) as ex:
            objs = list(ex.map(lambda kv: _compile(kv[0], [*kv[1], *_HOST_SANITIZE]), _SOURCES.items()))
        subprocess.check_call([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-Xarch_host", "-fsanitize=address",
                               "-Xarch_host", "-fsanitize=undefined", "-shared-libsan", *objs, "-o", LIB_PATH])
        return LIB_PATH
    finally:
        _OBJ, LIB_PATH = keep


def build_library(force: bool = True, jobs: int = 8) -> str:
    """Compile every HIP source and link libabsb.so (and the tests' libabsb_nowait.so).  `force=False` skips when up to date."""
    srcs = [os.path.join(_CSRC, n) for n in os.listdir(_CSRC)] + [os.path.join(_INCLUDE, "absb.h")]
    libs = (LIB_PATH, NOWAIT_PATH)
    if not force and all(os.path.exists(l) and os.path.getmtime(l) >= os.path.getmtime(s) for l in libs for s in srcs):
        return LIB_PATH
    os.makedirs(_OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        nowait = ex.submit(_compile, "build.hip", [*_SOURCES["build.hip"], "-DABSB_BUILD_WAIT_TICKS=1"], "build_nowait.o")
        objs = list(ex.map(lambda kv: _compile(*kv), _SOURCES.items()))
        other = [nowait.result() if name == "build.hip" else obj for name, obj in zip(_SOURCES, objs)]
    for lib, parts in zip(libs, (objs, other)):
        tmp = lib + f".tmp{os.getpid()}"
        subprocess.check_call([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *parts, "-o", tmp])
        os.replace(tmp, lib)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(force=True))
