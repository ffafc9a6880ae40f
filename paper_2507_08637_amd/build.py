"""Compile the HIP sources into libwersa.so next to this package (gfx950 only), and the autograd node into _wersa_torch.so."""
import os
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libwersa.so")
NODE = os.path.join(HERE, "_wersa_torch.so")
SOURCES = ["wersa_api.hip", "wersa_generic.hip", "wersa_profile.hip", "wersa_fast.hip",
           "wersa_block.hip", "wersa_split.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def node_command():
    """Host code against torch's headers: no device code in it."""
    import torch
    root = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    for inc in (root + "/include", root + "/include/torch/csrc/api/include", "/opt/rocm/include", sysconfig.get_paths()["include"]):
        cmd += ["-isystem", inc]
    return cmd + [os.path.join(CSRC, "wersa_torch.cpp"), "-o", NODE, "-L" + root + "/lib", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def build(verbose=False):
    """One object per source, compiled side by side with the autograd node, then one link."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory(prefix="wersa_build_") as tmp:
        def compile_one(src):
            obj = os.path.join(tmp, src.replace(".hip", ".o"))
            cmd = [hipcc] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj] if src.endswith(".hip") else node_command()
            if verbose:
                print(" ".join(cmd), flush=True)
            res = subprocess.run(cmd, capture_output=True, text=True)
            if res.returncode != 0:
                raise RuntimeError(f"compiler failed on {src}:\n" + res.stdout + res.stderr)
            return obj
        with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as pool:
            objs = list(pool.map(compile_one, SOURCES + ["wersa_torch.cpp"]))[:-1]
        cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("link failed:\n" + res.stdout + res.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
