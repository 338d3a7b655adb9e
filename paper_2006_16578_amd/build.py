"""Builds libbnn.so (HIP, gfx950 only) and _native.so (the binding's native module, host code) in-tree next to this file.

    python -m paper_2006_16578_amd.build [--force]

Each translation unit is compiled to an object in ``_build/`` and the objects are linked into
``libbnn.so``.  Objects are rebuilt when their source or any header is newer.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbnn.so")
NATIVE = os.path.join(HERE, "_native.so")
CXX = os.environ.get("CXX", "g++")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCES = ["bnn_api.hip", "bnn_valu.hip", "bnn_mfma.hip", "bnn_mfma_conv_v4.hip", "bnn_mfma_conv_v2.hip",
           "bnn_mfma_conv_v1.hip", "bnn_mfma_conv_v4_stream.hip", "bnn_mfma_conv_v2_stream.hip",
           "bnn_mfma_conv_v1_stream.hip", "bnn_mfma_conv_staged.hip", "bnn_aux.hip", "bnn_bwn.hip", "bnn_bwn_pixel.hip", "bnn_bwn_rect.hip", "bnn_fc_chain.hip", "bnn_persistent.hip", "bnn_probe.hip", "bnn_mfma_skinny.hip", "bnn_mfma_bits.hip", "bnn_mfma_signs.hip", "bnn_mfma_conv_patch.hip", "bnn_mfma_conv_xlds.hip", "bnn_mfma_conv_band.hip", "bnn_mfma_conv_taps.hip"]
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Wall", "-Wno-unused-value",
         "-Rpass-analysis=kernel-resource-usage",   # per-kernel register / scratch report, scanned for spills below
         # packed fp32 VALU forms are kept off for every device function of this library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _headers():
    hs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    hs.append(os.path.join(os.path.dirname(HERE), "include", "bnn.h"))
    return hs


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    srcp = os.path.join(CSRC, src)
    newest = max(os.path.getmtime(p) for p in [srcp] + _headers())
    if force or not os.path.exists(obj) or os.path.getmtime(obj) < newest:
        cmd = [HIPCC] + FLAGS + ["-c", srcp, "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        lines = r.stderr.splitlines()
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (src, "\n".join(l for l in lines if "remark:" not in l)))
        for l in lines:     # the resource-usage remarks are scanned below, not echoed
            if ("warning:" in l or "error:" in l) and "packed-fp32-ops" not in l and "target feature" not in l:
                sys.stderr.write(l + "\n")
        # a kernel that spills registers to scratch is a performance bug here: say so loudly
        name = "?"
        for l in lines:
            if "Function Name:" in l:
                name = l.split("Function Name:")[1].split("[")[0].strip()
            elif "VGPRs Spill:" in l and int(l.split("VGPRs Spill:")[1].split("[")[0]) > 0:
                sys.stderr.write("build.py: WARNING %s: kernel %s spills %s VGPRs\n"
                                 % (src, name, l.split("VGPRs Spill:")[1].split("[")[0].strip()))
    return obj


def _compile_native(force: bool) -> None:
    """The binding's native module: compiled against torch's headers, resolved against the torch that the process has loaded."""
    import sysconfig

    import torch

    from .binding import _native_stamp
    src = os.path.join(CSRC, "bnn_python.cpp")
    root = os.path.dirname(torch.__file__)
    cmd = [CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-I" + sysconfig.get_paths()["include"], "-I" + os.path.join(root, "include"),
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), '-DBNN_BUILT_FOR="%s"' % _native_stamp(), src,
           "-L" + os.path.join(root, "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python"]
    # rebuilt when a source is newer, and when the command differs: another torch or interpreter
    made_by = os.path.join(OBJ, "_native.cmd")
    newest = max(os.path.getmtime(p) for p in [src] + _headers())
    if not force and os.path.exists(NATIVE) and os.path.getmtime(NATIVE) >= newest and os.path.exists(made_by) and open(made_by).read() == repr(cmd):
        return
    tmp = NATIVE + ".tmp.%d" % os.getpid()
    subprocess.check_call(cmd + ["-o", tmp])
    os.replace(tmp, NATIVE)
    with open(made_by, "w") as f:
        f.write(repr(cmd))


def build(force: bool = False, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        native = ex.submit(_compile_native, force)
        objs = list(ex.map(lambda s: _compile(s, force), SOURCES))
        native.result()
    if force or not os.path.exists(LIB) or any(os.path.getmtime(o) > os.path.getmtime(LIB) for o in objs):
        tmp = LIB + ".tmp.%d" % os.getpid()
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
        os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
