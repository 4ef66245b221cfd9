"""Builds the HIP library (gfx950) in-tree: python -m paper_2605_18739_amd.build

Every source is compiled to an object of its own, side by side (the GEMM tile shapes are separate
translation units for this), and the objects are linked into libnvfp4_hip.so next to this file.
The binding's host code (_host.*.so, against torch's and Python's headers) is compiled beside them and linked to it."""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libnvfp4_hip.so")
HOST = os.path.join(HERE, "_host" + sysconfig.get_config_var("EXT_SUFFIX"))       # (tied to this Python by its name, to this torch by a check)
SOURCES = ["nvfp4_gemm_tile_256x256.hip", "nvfp4_gemm_tile_256x192.hip", "nvfp4_gemm_tile_128x128.hip",
           "nvfp4_gemm_split.hip", "nvfp4_quantize.hip", "nvfp4_quantize_resident.hip", "nvfp4_gemm.hip", "nvfp4_probe.hip", "nvfp4_api.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # packed-FP32 instructions are kept out of every kernel
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in proc.stdout.splitlines() if "is not a recognized feature" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)


def _host_commands():
    import torch
    root = os.path.dirname(torch.__file__)
    include = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
               sysconfig.get_paths()["include"]]
    obj = os.path.join(OBJ, "nvfp4_host.o")
    compile_ = (["g++", "-O2", "-std=c++17", "-fPIC", "-DNDEBUG", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
                + [a for d in include for a in ("-isystem", d)] + ["-c", os.path.join(CSRC, "nvfp4_host.cpp"), "-o", obj])
    link = ["g++", "-shared", obj, "-o", HOST, "-L" + HERE, "-l:" + os.path.basename(LIB), "-L" + os.path.join(root, "lib"),
            "-lc10", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN"]
    return compile_, link


def build(verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    objs = [os.path.join(OBJ, s.replace(".hip", ".o")) for s in SOURCES]
    host_compile, host_link = _host_commands()
    commands = [["hipcc"] + FLAGS + ["-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)] + [host_compile]
    jobs = max(1, min(len(commands), 16, int(os.environ.get("MAX_JOBS", os.cpu_count() or 4))))
    with ThreadPoolExecutor(jobs) as pool:
        list(pool.map(lambda c: _run(c, verbose), commands))
    _run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB], verbose)
    _run(host_link, verbose)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
