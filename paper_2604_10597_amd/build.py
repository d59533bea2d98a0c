"""Compile libcorey.so for gfx950 and its torch extension (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcorey.so")
NATIVE = os.path.join(HERE, "_native.so")          # Python extension: marshals torch tensors into libcorey
# the scan's kernels in several translation units: they compile side by side (the longest first)
SOURCES = [f"corey_scan_any_{t}_w{w}.hip" for t in ("bf16", "f16", "f32") for w in (3, 4)] + [
    "corey_scan_bf16.hip", "corey_scan_f16.hip", "corey_scan_f32.hip", "corey_conv.hip", "corey_entropy.hip", "corey_table.hip",
    "corey_decode.hip", "corey_scan.hip", "corey_host.cpp"]

# Packed-FP32 instruction selection is switched off for all device code (plain fp32 VALU ops only).
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def build_native(verbose: bool = False) -> str:
    """The torch extension: host code only, by the host compiler against torch's headers."""
    import torch
    t = os.path.dirname(torch.__file__)
    inc = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"), os.path.join(ROOT, "include"),
           sysconfig.get_paths()["include"]]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",
           *(a for i in inc[:2] for a in ("-isystem", i)), *(f"-I{i}" for i in inc[2:]), "-isystem", "/opt/rocm/include",
           os.path.join(CSRC, "corey_torch.cpp"), f"-L{os.path.join(t, 'lib')}", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip",
           "-ltorch_python", "-o", NATIVE]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return NATIVE


def build_lib(verbose: bool = False, extra: list[str] | None = None, jobs: int = 8) -> str:
    """Always recompiles the library and the torch extension; returns the path of the library."""
    cc = hipcc()
    inc = [f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}"]
    with tempfile.TemporaryDirectory(prefix="corey_build_") as tmp:
        def compile_one(src: str) -> str:
            obj = os.path.join(tmp, os.path.splitext(src)[0] + ".o")
            cmd = [cc, *HIPCC_FLAGS, "-x", "hip", *inc, *(extra or []), "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        with ThreadPoolExecutor(max_workers=max(1, jobs)) as pool:
            native = pool.submit(build_native, verbose)
            objs = list(pool.map(compile_one, SOURCES))
            native.result()
        link = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", "-Wno-unused-command-line-argument", *objs,
                "-o", LIB]
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.run(link, check=True)
    return LIB


if __name__ == "__main__":
    print(build_lib(verbose=True))
