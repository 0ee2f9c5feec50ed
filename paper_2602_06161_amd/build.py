"""Build the COVER HIP library for gfx950 (in-tree, hipcc).

Produces ``paper_2602_06161_amd/lib/libcover.so`` and the binding's native part,
``lib/_cover_host.so``, from ``csrc/``.  Run as
``python -m paper_2602_06161_amd.build``; ``__graft_entry__.build()`` calls ``build()``.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJDIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "lib", "libcover.so")
# the same library with the attention kernel's phase timestamps compiled in (measurement only)
LIB_TIMING = os.path.join(PKG, "lib", "libcover_timing.so")

# the Python binding's native part (host code against torch's headers)
HOST = os.path.join(PKG, "lib", "_cover_host.so")

ARCH = "gfx950"
HIPCC = os.environ.get("HIPCC") or shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

COMMON = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 VALU instructions stay off: plain fp32 ops only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", INCLUDE, "-I", CSRC,
]
# per-source extra flags
SOURCES = {
    "api.cpp": ["-x", "hip"],
    "cover_attn.hip": [],
    "cover_attn_w4.hip": [],
    "cover_attn_rect.hip": [],
    "cover_debug.hip": [],
    "cover_decode.hip": [],
    "cover_select.hip": ["-ffp-contract=off"],  # the selection is bit-exact fp64
    "cover_stats.hip": [],
    "cover_sample.hip": [],
}


# sources compiled a second time, with these flags, for LIB_TIMING
TIMING = {"cover_attn_w4.hip": ["-DCOVER_ATTN_TIMING=1"], "cover_attn_rect.hip": ["-DCOVER_RECT_TIMING=1"]}
# sources of LIB_TIMING only (the MFMA-counter calibration kernel)
TIMING_ONLY = {"cover_calib.hip": []}


def _compile(src: str, timing: bool = False) -> str:
    obj = os.path.join(OBJDIR, src + (".timing.o" if timing else ".o"))
    flags = SOURCES[src] if src in SOURCES else TIMING_ONLY[src]
    extra = TIMING.get(src, []) if timing else []
    cmd = [HIPCC, *COMMON, *flags, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def _build_host() -> None:
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    rocm = os.path.dirname(os.path.dirname(os.path.realpath(HIPCC)))
    tmp = HOST + ".tmp"
    cmd = [HIPCC, "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", INCLUDE, "-I", sysconfig.get_paths()["include"], "-I", os.path.join(rocm, "include")]
    for path in cpp_extension.include_paths():
        cmd += ["-I", path]
    cmd += [os.path.join(CSRC, "host.cpp"), "-o", tmp]
    for path in cpp_extension.library_paths():
        cmd += ["-L", path]
    cmd += ["-lc10", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for host.cpp:\n{' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, HOST)


def build(verbose: bool = True) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    os.makedirs(os.path.dirname(LIB), exist_ok=True)
    jobs = ([(src, False) for src in SOURCES] + [(src, True) for src in TIMING]
            + [(src, True) for src in TIMING_ONLY])
    with ThreadPoolExecutor(max_workers=len(jobs) + 1) as ex:
        host = ex.submit(_build_host)
        built = dict(zip(jobs, ex.map(lambda j: _compile(*j), jobs)))
        host.result()
    plain = [built[(src, False)] for src in SOURCES]
    timed = [built[(src, src in TIMING)] for src in SOURCES] + [built[(src, True)] for src in TIMING_ONLY]
    for lib, objs in ((LIB, plain), (LIB_TIMING, timed)):
        tmp = lib + ".tmp"
        cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
        os.replace(tmp, lib)
        if verbose:
            print(f"built {lib}", file=sys.stderr)
    if verbose:
        print(f"built {HOST}", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build()
