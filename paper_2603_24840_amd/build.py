"""Builds libarrol.so (HIP, gfx950 only) with hipcc and the binding's C++ marshalling (_marshal.so) with g++, in-tree.

    python -m paper_2603_24840_amd.build
"""
import os
import shlex
import shutil
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_DIR = os.path.join(HERE, "lib")
LIB_PATH = os.path.join(LIB_DIR, "libarrol.so")
MARSHAL_PATH = os.path.join(LIB_DIR, "_marshal.so")
SOURCES = ["score.hip", "score_mlp.hip", "train.hip", "select.hip", "compact.hip", "logprob.hip", "vote.hip", "confidence.hip", "grpo.hip", "policy.hip", "probe.hip", "api.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc_path():
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the ARRoL library can only be built with the ROCm toolchain")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if verbose and out.strip():
        print(out, flush=True)
    if res.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (os.path.basename(cmd[0]), out))


def build_marshal(verbose=True):
    """_marshal.so, with g++ (or $CXX) against torch's headers; what was there is gone if that fails."""
    import torch
    from .binding import built_for
    if os.path.exists(MARSHAL_PATH):
        os.remove(MARSHAL_PATH)
    t = os.path.dirname(torch.__file__)
    _run(shlex.split(os.environ.get("CXX") or "g++") +
         ["-O2", "-fPIC", "-shared", "-std=c++17", "-Wall", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
          '-DARROL_BUILT_FOR="%s"' % built_for(), "-D__HIP_PLATFORM_AMD__=1", "-I", os.path.join(ROOT, "include"),
          "-isystem", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc_path()))), "include"),
          "-isystem", os.path.join(t, "include"), "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
          "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL_PATH, "-L", LIB_DIR, "-larrol",
          "-L", os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10",
          "-Wl,-rpath,$ORIGIN", "-Wl,-z,now"], verbose)      # a symbol that another torch lacks is missed on loading, not in a call


def build(verbose=True):
    """The library, and the marshalling, without which it works as well: where that does not compile (no g++, no headers of
    Python or torch) a warning says so."""
    os.makedirs(LIB_DIR, exist_ok=True)
    _run([hipcc_path()] + HIPCC_FLAGS + ["-I", os.path.join(ROOT, "include"), "-I", CSRC] + [os.path.join(CSRC, s) for s in SOURCES] +
         ["-o", LIB_PATH], verbose)
    try:
        build_marshal(verbose)
    except (RuntimeError, OSError) as e:
        warnings.warn("built without _marshal.so: %s" % e, RuntimeWarning)
    return LIB_PATH


if __name__ == "__main__":
    build()
    sys.exit(0)
