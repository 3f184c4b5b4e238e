"""Build libmquant.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

hipcc cross-compiles without a GPU.  Flags: no FMA contraction and no
fast-math, so the fp32 butterflies and the quantizer multiply are single IEEE
operations; packed-fp32 instructions are switched off.
"""
import hashlib
import os
import shlex
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_DIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIB_DIR, "libmquant.so")
SOURCES = ["aifs.hip", "hadamard_quant.hip", "w4a8_gemm.hip", "w4a8_gemv.hip", "w4a8_sliced.hip", "w4a8_wide.hip", "w4a8_small.hip", "w4a8_walk.hip", "attention.hip",
           "w4g128_gemm.hip", "w4g128_walk.hip"]
# The benchmark's measurement probes: their own shared object, outside the product's ABI.
PROBES_LIB = os.path.join(LIB_DIR, "libmquant_probes.so")
PROBES_SOURCES = ["probes.hip"]
# The interpreter's short way to the library's launches: a CPython module without device code, under the name that
# this interpreter's ABI gives its modules.  Calls go through ctypes where it is not built.
CALL_LIB = os.path.join(LIB_DIR, "mquant_fastcall" + sysconfig.get_config_var("EXT_SUFFIX"))
CALL_SOURCES = ["fastcall.c"]
HEADERS = ["mquant_internal.h", "hadamard_segment.h", "w4a8_common.h", "w4g128_common.h", "lds_dma.h", "probes.h"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter", "-Wno-inline-asm",
]
CC_FLAGS = ["-O2", "-std=gnu11", "-fPIC", "-shared", "-Wall"]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def _deps(srcs):
    headers = [] if srcs is CALL_SOURCES else HEADERS
    return ([os.path.join(CSRC, s) for s in srcs] + [os.path.join(CSRC, h) for h in headers]
            + [os.path.join(ROOT, "include", "mquant.h")])


def source_hash(srcs=None) -> str:
    """Hash of the sources, headers and compiler flags a library is built from, for the call module
    of the interpreter's ABI too.  It is compiled into libmquant.so (mquant_build_id) and written
    next to each library, so that staleness is judged by content: file times do not survive every
    copy of the tree."""
    flags = CC_FLAGS + [sysconfig.get_config_var("SOABI")] if srcs is CALL_SOURCES else HIPCC_FLAGS
    h = hashlib.sha256(" ".join(flags).encode())
    for d in _deps(SOURCES if srcs is None else srcs):
        h.update(os.path.basename(d).encode())
        with open(d, "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def _stale(lib, srcs) -> bool:
    if not os.path.exists(lib) or not os.path.exists(lib + ".id"):
        return True
    with open(lib + ".id") as f:
        return f.read().strip() != source_hash(srcs)


def _cc():
    return shlex.split(os.environ.get("CC") or "gcc")


def _can_build_call() -> bool:
    return shutil.which(_cc()[0]) is not None and os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h"))


def _call_stale() -> bool:
    """The call module can be done without, but not be another build's."""
    return _stale(CALL_LIB, CALL_SOURCES) and (os.path.exists(CALL_LIB) or _can_build_call())


def _hip_stale() -> bool:
    return _stale(LIB, SOURCES) or _stale(PROBES_LIB, PROBES_SOURCES)


def is_stale() -> bool:
    """True when a library is missing or was built from other sources, headers or flags."""
    return _hip_stale() or _call_stale()


def _compile(lib, srcs, verbose):
    build_id = source_hash(srcs)
    if srcs is CALL_SOURCES:
        cmd = [*_cc(), *CC_FLAGS, "-I", sysconfig.get_paths()["include"]]
    else:
        cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *HIPCC_FLAGS, f'-DMQUANT_BUILD_ID="{build_id}"', "-I", CSRC]
    cmd += ["-I", os.path.join(ROOT, "include"), *[os.path.join(CSRC, s) for s in srcs], "-o", lib]
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass prints a harmless "not a recognized feature" line per file
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + out)
    if verbose and out.strip():
        print(out)
    with open(lib + ".id", "w") as f:
        f.write(build_id + "\n")


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile libmquant.so, libmquant_probes.so and the call module; with force=False only what is stale."""
    os.makedirs(LIB_DIR, exist_ok=True)
    if force or _stale(LIB, SOURCES):
        _compile(LIB, SOURCES, verbose)
    if force or _stale(PROBES_LIB, PROBES_SOURCES):
        _compile(PROBES_LIB, PROBES_SOURCES, verbose)
    if (force or _stale(CALL_LIB, CALL_SOURCES)) and _can_build_call():
        _compile(CALL_LIB, CALL_SOURCES, verbose)
    elif _call_stale():
        os.remove(CALL_LIB)                          # of other sources, and nothing here to build it with
    return LIB


def ensure_fresh() -> str:
    """What tests, the smoke run and the benchmark call before loading the library: rebuild
    when the sources differ from what the binary was built from, so an edited kernel is never
    checked against an older build.  Where no compiler is present a stale library is an error."""
    if _hip_stale() and not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")):
        raise RuntimeError("libmquant.so is missing or stale and there is no hipcc to build it")
    if is_stale():
        build(force=False)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
