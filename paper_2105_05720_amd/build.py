"""Builds libccfused.so for gfx950 with hipcc, in-tree (next to this file).

The library is several translation units (one per kernel family) only so that they compile side by side; each is
compiled to an object file and the objects are linked into one shared library, whose dynamic symbol table is cut down
to the C ABI by csrc/exports.map.  Beside it, with g++, the extension module through which Python's step calls reach it,
if this Python's headers are there: nothing but time depends on it."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
SOURCES = [os.path.join(CSRC, n) for n in ("ccfused.hip", "launch_adam_f16.hip", "launch_adam_f32.hip", "launch_lamb.hip", "launch_lamb_one.hip",
                                           "launch_unfused.hip")]
EXPORTS_MAP = os.path.join(CSRC, "exports.map")
DEPS = SOURCES + [os.path.join(CSRC, "kernels.hip.h"), os.path.join(CSRC, "plan.hpp"), os.path.join(CSRC, "piece_order.hpp"),
                  os.path.join(CSRC, "cache_rules.hpp"), os.path.join(CSRC, "meeting.hpp"), os.path.join(CSRC, "flag_word.hpp"), os.path.join(CSRC, "packed_args.hpp"), os.path.join(CSRC, "tuning.hpp"), os.path.join(CSRC, "occupancy.hpp"),
                  os.path.join(CSRC, "launch_adam.inc.hpp"),
                  os.path.join(ROOT, "include", "ccfused.h"), EXPORTS_MAP]
LIB = os.path.join(_HERE, "libccfused.so")
STEP_CALLS_SOURCE = os.path.join(CSRC, "step_calls.cpp")
# A module of CPython's, for the Python that builds it; host code only.
STEP_CALLS = os.path.join(_HERE, "_step_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
OBJ_DIR = os.path.join(_HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-fvisibility=hidden",
    "-ffp-contract=off",                                              # fused multiply-adds are written out by hand
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",      # no packed-fp32 instructions
    # The kernels issue their counting atomics (flag count, chunk ticket) early and look at the result a block of work
    # later.  The compiler's wave-level atomic aggregation would rewrite each into "one lane adds, readfirstlane the
    # result", which needs the result at once and so drains the wave's memory counter right behind the atomic.
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _older(built, sources) -> bool:
    return not os.path.exists(built) or any(os.path.getmtime(d) > os.path.getmtime(built) for d in sources)


def is_stale() -> bool:
    return _older(LIB, DEPS)


def build_step_calls():
    """The extension module; without a compiler or Python's headers None, and the step calls go the way through ctypes."""
    tmp = STEP_CALLS + ".tmp%d" % os.getpid()
    try:
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wextra", "-Wno-cast-function-type",
                               "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), "-o", tmp, STEP_CALLS_SOURCE])
    except (OSError, subprocess.CalledProcessError) as e:
        print("the step calls' extension module was not built (%s); they take 1 to 2 us longer without it" % e, file=sys.stderr)
        if os.path.exists(STEP_CALLS):
            os.remove(STEP_CALLS)             # of other sources
        return None
    os.replace(tmp, STEP_CALLS)
    return STEP_CALLS


def build_library(force: bool = True, extra=()) -> str:
    """Compile the HIP library and the extension module.  force=False skips what is newer than its sources."""
    if force or _older(STEP_CALLS, [STEP_CALLS_SOURCE, os.path.join(ROOT, "include", "ccfused.h")]):
        build_step_calls()
    if not force and not is_stale():
        return LIB
    os.makedirs(OBJ_DIR, exist_ok=True)
    tag = ".%d" % os.getpid()
    objs = [os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + tag + ".o") for src in SOURCES]

    def compile_one(pair):
        src, obj = pair
        subprocess.check_call([HIPCC] + FLAGS + list(extra) + ["-c", "-o", obj, src])
    try:
        with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as pool:
            list(pool.map(compile_one, zip(SOURCES, objs)))
        tmp = LIB + ".tmp%d" % os.getpid()
        subprocess.check_call([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-Wl,--version-script=" + EXPORTS_MAP,
                               "-o", tmp] + objs)
        os.replace(tmp, LIB)
    finally:
        for obj in objs:
            if os.path.exists(obj):
                os.remove(obj)
    return LIB


if __name__ == "__main__":
    print(build_library(force=True, extra=sys.argv[1:]))
