"""Compile the gfx950 kernels and the C-ABI host code into paper_2511_12653_amd/libfq.so.

hipcc cross-compiles for gfx950 without a GPU.  Flags: IEEE arithmetic only (no fast-math, no
implicit FMA contraction -- the kernels call fma explicitly where they want one) and no packed
FP32 instructions.  The first 14 dwords of a kernel's scalar arguments (all that fit beside the address of the
rest) come in registers with the launch instead of being loaded by every wavefront.

The binding's native calls (csrc/fq_call.c) go into a CPython extension next to the library, by the host's C compiler.
"""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfq.so")
SOURCES = [os.path.join(CSRC, f) for f in ("fq_kernels.hip", "fq_distill.hip", "fq_api.cpp")]
CALL_SOURCE = os.path.join(CSRC, "fq_call.c")
CALL = os.path.join(HERE, "_fqcall" + sysconfig.get_config_var("EXT_SUFFIX"))
CC = os.environ.get("CC", "gcc")
HEADERS = [os.path.join(CSRC, "fq_internal.h"), os.path.join(CSRC, "fq_device.h"),
           os.path.join(HERE, "..", "include", "fq.h")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
         "-fno-fast-math", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=14", "-Wall", "-Wextra", "-Wno-unused-command-line-argument"]


def stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(CALL):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(CALL))
    return any(os.path.getmtime(p) > t for p in SOURCES + HEADERS + [CALL_SOURCE])


def build(force: bool = True, extra=()) -> str:
    if not force and not stale():
        return LIB
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [HIPCC, *FLAGS, *extra, "-I", os.path.join(HERE, "..", "include"), *SOURCES, "-o", tmp]
    # The packed-FP32 switch is a gfx950 target feature.  hipcc hands -Xclang options to the host
    # pass as well (it offers no way to give one to the device pass alone), where x86-64 answers
    # "not a recognized feature for this target (ignoring feature)" once per source and pass: drop
    # exactly those lines and show everything else the compiler says.
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    noise = ("'-packed-fp32-ops' is not a recognized feature for this target", "warning generated when compiling for host",
             "warnings generated when compiling for host")
    kept = [ln for ln in p.stdout.splitlines() if not any(n in ln for n in noise)]
    if kept:
        print("\n".join(kept), file=sys.stderr)
    if p.returncode != 0:
        raise subprocess.CalledProcessError(p.returncode, cmd)
    os.replace(tmp, LIB)
    build_call()
    return LIB


def build_call() -> str:
    """The extension; it finds the library in its own folder."""
    tmp = CALL + ".tmp.%d" % os.getpid()
    subprocess.run([CC, "-O2", "-std=c11", "-fPIC", "-shared", "-Wall", "-Wextra", "-Wno-missing-field-initializers",
                    "-I", sysconfig.get_paths()["include"], CALL_SOURCE, "-L", HERE, "-l:libfq.so", "-Wl,-rpath,$ORIGIN",
                    "-o", tmp], check=True)
    os.replace(tmp, CALL)
    return CALL


def ensure_built() -> str:
    """Build only if no library is there (tests, smoke and bench load what is built)."""
    return LIB if os.path.exists(LIB) and os.path.exists(CALL) else build(force=True)


if __name__ == "__main__":
    print(build())
