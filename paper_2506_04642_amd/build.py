"""Compile libtadakv.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtadakv.so")

# packed-fp32 instruction forms are switched off for every device translation unit
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# matrix-instruction results go straight to ordinary vector registers; the direct-to-LDS fetches
# are issued by hand and name M0 as clobbered, which the compiler remarks on at every use
# (the assembly text is kept next to the object and read by verify_hand_loads after the compile)
MFMA = ["-mllvm", "-amdgpu-mfma-vgpr-form", "-Wno-inline-asm", "-save-temps=obj"]
# (source, extra flags, object folder below _build): the quantiser is compiled without fused multiply-add contraction so
# that every binary32 operation rounds once, in the order written; the split kernel's units compile side by side
UNITS = [
    ("decode_mfma.hip", MFMA + ["-DTADA_KEY_BITS=8"], "k8"),
    ("decode_mfma.hip", MFMA + ["-DTADA_KEY_BITS=4"], "k4"),
    ("decode_mfma.hip", MFMA + ["-DTADA_KEY_BITS=2"], "k2"),
    ("decode_mfma.hip", MFMA + ["-DTADA_KEY_BITS=8", "-DTADA_STREAM=1"], "k8s"),
    ("decode_mfma.hip", MFMA + ["-DTADA_KEY_BITS=4", "-DTADA_STREAM=1"], "k4s"),
    ("decode_mfma.hip", MFMA + ["-DTADA_KEY_BITS=2", "-DTADA_STREAM=1"], "k2s"),
    ("tadakv_abi.cpp", ["-x", "hip"], ""),
    ("quant_append.hip", ["-ffp-contract=off"], ""),
    ("compressv.hip", ["-ffp-contract=off", "-mllvm", "-amdgpu-mfma-vgpr-form", "-save-temps=obj"], ""),
    ("decode_valu.hip", [], ""),
    ("decode_mfma_host.cpp", ["-x", "hip"], ""),
    ("decode_raw.hip", ["-mllvm", "-amdgpu-mfma-vgpr-form"], ""),
    ("xhead_dense.hip", [], ""),
    ("stream_probe.hip", [], ""),
]


def sources():
    return [os.path.join(CSRC, s) for s in dict.fromkeys(u[0] for u in UNITS)] + [
        os.path.join(CSRC, "tadakv_internal.h"),
        os.path.join(CSRC, "quant_wave.h"),
        os.path.join(CSRC, "join.h"),
        os.path.join(os.path.dirname(HERE), "include", "tadakv.h"),
    ]


def build_library(force: bool = True, verbose: bool = False) -> str:
    """Compile every translation unit and link the shared library.  With force=False an
    up-to-date library is kept."""
    if not force and os.path.exists(LIB):
        if all(os.path.getmtime(LIB) >= os.path.getmtime(s) for s in sources()):
            return LIB
    objdir = os.path.join(HERE, "_build")
    objs = []
    procs = []
    for src, extra, sub in UNITS:
        os.makedirs(os.path.join(objdir, sub), exist_ok=True)
        obj = os.path.join(objdir, sub, os.path.splitext(src)[0] + ".o")
        cmd = ["hipcc"] + COMMON + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for cmd, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            raise RuntimeError("hipcc failed: %s\n%s" % (" ".join(cmd), out))
        if verbose and out.strip():
            print(out)
    # the kernels that issue loads by hand: the compiler must have left the destinations alone, and the order of counted fetches
    import importlib.util

    spec = importlib.util.spec_from_file_location("verify_hand_loads", os.path.join(HERE, "verify_hand_loads.py"))
    _v = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(_v)  # (by path: this file also runs as a script)

    hand = [("decode_mfma", k, "decode_split_mfma_kernel", True) for k in ("k2", "k4", "k8", "k2s", "k4s", "k8s")] + [("compressv", "", "compressv_gemm_kernel", False)]
    for unit, sub, kernel, glob in hand:
        here = os.path.join(objdir, sub)
        checked = _v.verify(os.path.join(here, unit + "-hip-amdgcn-amd-amdhsa-gfx950.s"), kernel, glob)
        if verbose:
            print("verify_hand_loads: %s: %d kernels, %d global requests, %d LDS reads" % ((os.path.join(sub, unit),) + checked))
        if unit == "compressv":
            _v.verify_fetch_order(os.path.join(here, unit + "-hip-amdgcn-amd-amdhsa-gfx950.s"))
        for f in os.listdir(here):
            if f.startswith(unit + "-") or f.startswith(unit + ".hip-"):
                os.remove(os.path.join(here, f))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
