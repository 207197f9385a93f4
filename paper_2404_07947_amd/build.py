"""Builds libexe.so (HIP kernels + runtime + C ABI) for gfx950 with hipcc, and _call (Python's way to its serving calls), in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libexe.so")
# csrc/call.c: host code against Python's headers, named for the Python that it is built for
CALL = os.path.join(HERE, "_call" + sysconfig.get_config_var("EXT_SUFFIX"))
CC = os.environ.get("CC", "gcc")
SOURCES = ["kernels_elementwise.hip", "kernels_gemm.hip", "kernels_gemm_large.hip", "kernels_gemm_stream.hip", "kernels_gemm_f32.hip", "kernels_attn.hip", "kernels_small.hip", "runtime.hip", "probe.hip", "sched.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# Kernel arguments preloaded into scalar registers instead of fetched by each wave's first instructions: decode iterations of
# small models run 1-3 % faster (0.3 us of a 4-6 us launch).
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-mllvm", "-amdgpu-kernarg-preload-count=16",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _headers_mtime() -> float:
    hs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    inc = os.path.join(HERE, "..", "include")
    hs += [os.path.join(inc, f) for f in os.listdir(inc) if f.endswith(".h")]
    return max(os.path.getmtime(h) for h in hs)


def build(force: bool = False, verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    hm = _headers_mtime()

    def compile_one(src: str) -> str:
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
        if not force and os.path.exists(o) and os.path.getmtime(o) >= max(os.path.getmtime(s), hm):
            return o
        cmd = [HIPCC, *FLAGS, "-c", s, "-o", o]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                         if "packed-fp32-ops" not in l and l.strip())
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{msgs}")
        if msgs and verbose:
            print(msgs, flush=True)
        return o

    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    if force or not os.path.exists(LIB) or any(os.path.getmtime(o) > os.path.getmtime(LIB) for o in objs):
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB + ".tmp", *objs]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        os.replace(LIB + ".tmp", LIB)
    src = os.path.join(CSRC, "call.c")
    if force or not os.path.exists(CALL) or os.path.getmtime(src) > os.path.getmtime(CALL):
        cmd = [CC, "-O2", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"], src, "-o", CALL + ".tmp"]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        os.replace(CALL + ".tmp", CALL)
    return LIB


def build_variant(tag: str, defines, verbose: bool = True) -> str:
    """Builds libexe_<tag>.so: the library with the tile GEMMs compiled as a measurement variant (defines such as
    -DEXE_GEMM_ABLATE=1, see csrc/gemm_tile.h, or -DEXE_GEMM_ISSUE_AT=1, see csrc/kernels_gemm.hip; an ablated variant's
    results are meaningless, its timing isolates a part of the kernel).  The other objects are the library's own."""
    build(verbose=verbose)
    objs = []
    for src in SOURCES:
        obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
        if src in ("kernels_gemm.hip", "kernels_gemm_large.hip"):
            obj = obj[:-2] + f"_{tag}.o"
            cmd = [HIPCC, *FLAGS, *defines, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            r = subprocess.run(cmd, capture_output=True, text=True)
            if r.returncode != 0:
                raise RuntimeError("hipcc failed:\n" + "\n".join(l for l in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in l))
        objs.append(obj)
    lib = os.path.join(HERE, f"libexe_{tag}.so")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs], check=True)
    return lib


if __name__ == "__main__":
    if "--variant" in sys.argv:
        print(build_variant(sys.argv[sys.argv.index("--variant") + 1], [a for a in sys.argv if a.startswith("-D")]))
    else:
        build(force="--force" in sys.argv)
