"""Compile the HIP sources of the LAQ library for gfx950, and the Python binding of its hot calls, into in-tree
shared objects."""
from __future__ import annotations

import glob
import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "liblaq.so")
NATIVE = os.path.join(PKG, "_native.so")          # the binding of the calls in a model's loop

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # let MFMA results land in ordinary VGPRs: the softmax consumes them directly
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def needs_build() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(NATIVE):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(NATIVE))
    deps = sources() + glob.glob(os.path.join(CSRC, "*.cpp")) + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    return any(os.path.getmtime(f) > t for f in deps)


def build(force: bool = True, verbose: bool = False) -> str:
    """Run hipcc (cross-compiles without a GPU): every source to an object file, side by side, then one
    link.  Returns the path of the library."""
    if not force and not needs_build():
        return LIB
    from concurrent.futures import ThreadPoolExecutor
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    include = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]

    def run(cmd):
        res = subprocess.run(cmd, capture_output=True, text=True)
        if verbose or res.returncode != 0:
            print(res.stdout)
            print("\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l))
        if res.returncode != 0:
            raise RuntimeError("hipcc failed (exit %d): %s" % (res.returncode, " ".join(cmd[-3:])))

    def compile_one(src):
        obj = os.path.join(objdir, os.path.basename(src)[:-4] + ".%d.o" % os.getpid())
        run([hipcc] + compile_flags + include + ["-c", "-o", obj, src])
        return obj

    def compile_native():
        # host code only: CPython and torch headers, no GPU code (torch's libraries are in the process that loads it)
        import sysconfig

        import torch
        from torch.utils.cpp_extension import include_paths, library_paths
        tmp = NATIVE + ".tmp.%d" % os.getpid()
        try:
            run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-missing-field-initializers",
                 "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-I", os.path.join(ROOT, "include")]
                + ["-isystem" + p for p in include_paths()] + ["-isystem" + sysconfig.get_paths()["include"]]
                + [os.path.join(CSRC, "laq_native.cpp")] + ["-L" + p for p in library_paths()]
                + ["-lc10", "-ltorch_cpu", "-ltorch_python", "-o", tmp])
            os.replace(tmp, NATIVE)
        finally:
            if os.path.exists(tmp):
                os.remove(tmp)

    with ThreadPoolExecutor(max_workers=min(8, len(sources()) + 1)) as pool:
        native = pool.submit(compile_native)
        objs = list(pool.map(compile_one, sources()))
    tmp = LIB + ".tmp.%d" % os.getpid()
    try:
        run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
        os.replace(tmp, LIB)
    finally:
        for o in objs:
            if os.path.exists(o):
                os.remove(o)
    native.result()                                # (the library is there even where its compiled binding does not build)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
