"""Compile the gfx950 kernels and the C-ABI host code into paper_2511_12653_amd/libfq.so.

hipcc cross-compiles for gfx950 without a GPU.  Flags: IEEE arithmetic only (no fast-math, no
implicit FMA contraction -- the kernels call fma explicitly where they want one) and no packed
FP32 instructions.  The first 14 dwords of a kernel's scalar arguments (all that fit beside the address of the
rest) come in registers with the launch instead of being loaded by every wavefront.

The binding's native calls (csrc/fq_call.c) go into a CPython extension next to the library, by the host's C compiler.
They only shorten the marshalling: where there is no compiler, or no headers of this interpreter, the library is built
without them and the binding's Python forms serve.
"""
import os
import shlex
import subprocess
import sys
import sysconfig
import tempfile

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
    # Both files are made in a folder beside their own and go there together: never a new library beside an old extension.
    with tempfile.TemporaryDirectory(prefix="build.", dir=os.path.dirname(LIB)) as made:
        lib = os.path.join(made, os.path.basename(LIB))
        _compile_library(lib, extra)
        call = _compile_call(made)
        if call is None and os.path.exists(CALL):
            os.remove(CALL)                            # made from the library before
        os.replace(lib, LIB)
        if call is not None:
            os.replace(call, CALL)
    return LIB


def _compile_library(to: str, extra) -> None:
    cmd = [HIPCC, *FLAGS, *extra, "-I", os.path.join(HERE, "..", "include"), *SOURCES, "-o", to]
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


def _compile_call(folder: str):
    """The extension, linked against the library in `folder` and made there; it will find the library in its own
    folder.  None, with a message, where it cannot be compiled."""
    to = os.path.join(folder, os.path.basename(CALL))
    cmd = [*shlex.split(CC), "-O2", "-std=c11", "-fPIC", "-shared", "-Wall", "-Wextra", "-Wno-missing-field-initializers",
           "-I", sysconfig.get_paths()["include"], CALL_SOURCE, "-L", folder, "-l:" + os.path.basename(LIB),
           "-Wl,-rpath,$ORIGIN", "-o", to]
    try:
        subprocess.run(cmd, check=True)
    except (OSError, subprocess.CalledProcessError) as e:
        print("no native calls, the binding goes through its Python forms: %s" % e, file=sys.stderr)
        return None
    return to


def build_call():
    """The extension alone, for the library that is there; returns its path, or None."""
    with tempfile.TemporaryDirectory(prefix="build.", dir=os.path.dirname(CALL)) as made:
        os.symlink(LIB, os.path.join(made, os.path.basename(LIB)))
        call = _compile_call(made)
        if call is None:
            return None
        os.replace(call, CALL)
    return CALL


def ensure_built() -> str:
    """Build only what is not there (tests, smoke and bench load what is built)."""
    if not os.path.exists(LIB):
        return build(force=True)
    if not os.path.exists(CALL):
        build_call()
    return LIB


if __name__ == "__main__":
    print(build())
