"""Builds libpatnufft.so in-tree with hipcc for gfx950.

Usage: ``python -m paper_0808_3510_amd.build`` (or ``build()`` from Python).
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpatnufft.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["plan.cpp", "capi.cpp", "general.hip", "linepair.hip", "transverse.hip", "kernels.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _compile(flags: list[str], lib: str, verbose: bool):
    """The sources side by side (each takes a minute or two), then one link."""
    tmp = tempfile.mkdtemp(prefix="build_", dir=HERE)
    try:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        runs = [subprocess.Popen([HIPCC, *flags, "-c", "-I" + os.path.join(ROOT, "include"), os.path.join(CSRC, s),
                                  "-o", o], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
                for s, o in zip(SOURCES, objs)]
        outs = [r.communicate()[0] for r in runs]
        failed = any(r.returncode != 0 for r in runs)
        if not failed:
            res = subprocess.run([HIPCC, *flags, "-shared", *objs, "-o", lib + ".tmp"], capture_output=True, text=True)
            outs.append(res.stdout + res.stderr)
            failed = res.returncode != 0
        if verbose or failed:
            sys.stderr.write("".join(outs))
        if failed:
            raise RuntimeError("hipcc failed building " + os.path.basename(lib))
        os.replace(lib + ".tmp", lib)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)


SAN_LIB = os.path.join(ROOT, "_build", "libpatnufft_hostsan.so")


def build_host_sanitized(verbose: bool = False) -> str:
    """The library with its host side (plan, C ABI, launchers) built with
    AddressSanitizer and UndefinedBehaviorSanitizer, for the CPU checks of the
    host logic.  Load it with the ASan runtime preloaded (``asan_runtime()``).
    Not for the GPU: its device code is built at -O1."""
    os.makedirs(os.path.dirname(SAN_LIB), exist_ok=True)
    # (device code at -O1 for a quick build; the sanitizers apply to the host
    # side only, each -fsanitize= behind -Xarch_host)
    _compile(["--offload-arch=gfx950", "-O1", "-g", "-std=c++17", "-fPIC",
              "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
              "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
              "-Xarch_host", "-fno-sanitize-recover=all", "-Xarch_host", "-fno-omit-frame-pointer",
              "-Xarch_host", "-shared-libsan"], SAN_LIB, verbose)
    return SAN_LIB


def asan_runtime() -> str:
    """Path of the compiler's shared ASan runtime (to preload)."""
    res = subprocess.run([HIPCC, "-print-file-name=libclang_rt.asan-x86_64.so"], capture_output=True, text=True)
    path = res.stdout.strip()
    if not os.path.isabs(path) or not os.path.exists(path):
        raise RuntimeError("ASan runtime not found")
    return path


def build(verbose: bool = False) -> str:
    _compile(FLAGS, LIB, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
