"""Build libtdc.so (HIP, gfx950) in-tree with hipcc.  ``python -m paper_2211_03715_amd.build``.

``python -m paper_2211_03715_amd.build --probes`` builds libtdc_probe.so instead: the same sources with phase
timestamps compiled in (a bring-up aid, see build_probes)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ_DIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libtdc.so")

SOURCES = ["tdc_api.hip", "tdc_pack.hip", "tdc_naive.hip", "tdc_gemm.hip", "tdc_tile.hip", "tdc_fused.hip", "tdc_chain.hip", "tdc_chain_mb1.hip", "tdc_chain_mb2.hip", "tdc_chain_mb4.hip",
           "tdc_chain3.hip", "tdc_chain3_nchw.hip", "tdc_chain3_runs.hip", "tdc_chain3_nhwc.hip",
           "tdc_chain_bf3.hip", "tdc_chain_bf3_nchw.hip", "tdc_chain_bf3_runs.hip", "tdc_chain_bf3_nhwc.hip", "tdc_pack_bf3.hip", "tdc_tile_bf3.hip",
           "tdc_fm.hip", "tdc_select.cpp", "tdc_ranks.cpp", "tdc_hosvd.cpp"]

# Packed-fp32 VALU instructions are switched off for every device translation unit.
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wall", "-Wno-unused-command-line-argument",
             "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc()] + HIP_FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if "warning" in warn:
        sys.stderr.write(warn + "\n")
    return obj


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared library.  Always recompiles."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


PROBE_LIB = os.path.join(PKG, "libtdc_probe.so")


def build_probes(verbose: bool = False) -> str:
    """Bring-up build with phase timestamps: libtdc_probe.so, the same sources compiled with -DTDC_PHASE_TIMING.

    The probe buffer is one device array shared by every kernel (tdc_mfma.h), so all sources go into ONE translation
    unit here; the shipped library is never built this way.  `python -m paper_2211_03715_amd.probes` reads the
    timestamps back."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    unity = os.path.join(OBJ_DIR, "tdc_probe_all.hip")
    with open(unity, "w") as f:
        f.write("// generated by build.py: every source of libtdc.so in one translation unit\n")
        for src in SOURCES:
            f.write('#include "%s"\n' % os.path.join(CSRC, src))
    tmp = PROBE_LIB + ".tmp%d" % os.getpid()
    cmd = [_hipcc()] + HIP_FLAGS + ["-DTDC_PHASE_TIMING", "-shared", unity, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for the probe build:\n%s\n%s" % (r.stdout, r.stderr))
    os.replace(tmp, PROBE_LIB)
    if verbose:
        print("built", PROBE_LIB)
    return PROBE_LIB


if __name__ == "__main__":
    if "--probes" in sys.argv[1:]:
        build_probes(verbose=True)
    else:
        build(verbose=True)
