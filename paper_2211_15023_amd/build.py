"""Compile in-tree: csrc/*.hip -> libaccerl.so (gfx950 only), csrc/arguments.cpp -> accerl_args.so (the binding's marshalling)."""
import glob
import importlib.util
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
SO = os.path.join(HERE, "libaccerl.so")
ARGS_SO = os.path.join(HERE, "accerl_args.so")
OBJ = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument", "-I", INCLUDE, "-I", CSRC]


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    r = subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    return obj, err


def build(verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        res = list(ex.map(_compile, srcs))
    if verbose:
        for _, err in res:
            if err.strip():
                print(err)
    objs = [o for o, _ in res]
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", SO, *objs],
                       capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("link failed:\n" + r.stderr)
    _build_args(verbose)
    return SO


def compile_module(src, out, extra=()):
    """A CPython module on torch's headers and libaccerl.so: host code, by the host's compiler.  Returns what the compiler said."""
    torch = os.path.dirname(importlib.util.find_spec("torch").origin)
    rocm = os.path.dirname(os.path.dirname(HIPCC)) if os.path.isabs(HIPCC) else "/opt/rocm"
    r = subprocess.run([CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-I", INCLUDE, *extra,
                        *(a for d in (f"{torch}/include", f"{torch}/include/torch/csrc/api/include", f"{rocm}/include",
                                      sysconfig.get_path("include")) for a in ("-isystem", d)),
                        src, "-o", out, "-L", HERE, "-l:libaccerl.so", "-L", f"{torch}/lib",
                        "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"], capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError(f"{os.path.basename(src)} failed:\n" + r.stderr)
    return r.stderr


def _build_args(verbose):
    """The module that takes torch tensors to pointers."""
    said = compile_module(os.path.join(CSRC, "arguments.cpp"), ARGS_SO)
    if verbose and said.strip():
        print(said)


if __name__ == "__main__":
    print(build(verbose=True))
