"""Build libbittrain.so for gfx950 with hipcc (cross-compiles without a GPU), and the binding's call module with g++."""
import importlib.util
import os
import re
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "csrc", "bittrain.hip")
LIB = os.path.join(HERE, "libbittrain.so")
# measurement aids for bench.py: the same kernels with per-tile time stamps compiled in, plus a plain stream
BENCH_SRC = os.path.join(HERE, "csrc", "bench_aids.hip")
BENCH_LIB = os.path.join(HERE, "libbittrain_bench.so")
# the calls on torch tensors, checked and marshalled in C++
CALL_SRC = os.path.join(HERE, "csrc", "call.cpp")
CALL_LIB = os.path.join(HERE, "_call.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
    # packed fp32 VALU forms are kept out of the device code: some of them have given wrong results
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build(verbose=False, extra_flags=(), lib=LIB, src=SRC):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + HIPCC_FLAGS + list(extra_flags) + ["-I", os.path.join(ROOT, "include"), src, "-o", lib]
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass warns that it does not know the packed-fp32 feature: harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    if lib == LIB:
        build_call(verbose)
    return lib


def build_bench_aids(verbose=False, extra_flags=()):
    return build(verbose=verbose, extra_flags=extra_flags, lib=BENCH_LIB, src=BENCH_SRC)


def build_call(verbose=False):
    torch = os.path.dirname(importlib.util.find_spec("torch").origin)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    with open(os.path.join(torch, "version.py")) as f:      # (the module tells which torch it was compiled with)
        version = re.search(r"^__version__\s*=\s*['\"]([^'\"]+)", f.read(), re.M).group(1)
    cmd = ["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           '-DBT_TORCH_VERSION="%s"' % version,
           "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(torch, "include"),
           "-isystem", os.path.join(torch, "include", "torch", "csrc", "api", "include"), "-isystem", os.path.join(rocm, "include"),
           CALL_SRC, "-o", CALL_LIB, "-L", os.path.join(torch, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    return CALL_LIB


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_bench_aids(verbose=True))
