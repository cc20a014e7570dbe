"""Build libspot.so (gfx950) in-tree with hipcc, and the Python binding's native
marshalling (_binding.so, host code against torch's headers) with g++.

    python -m paper_2606_22874_amd.build

Each HIP source is compiled to an object in ``_build/`` (in parallel), then
linked into ``paper_2606_22874_amd/libspot.so``.  Packed-FP32 instructions are
disabled for device code.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
SO = os.path.join(PKG, "libspot.so")
BINDING = os.path.join(PKG, "_binding.so")
ARCH = "gfx950"

SOURCES = ["api.hip", "frontend.hip", "frontend_mfma.hip", "score.hip", "score_many.hip", "score_tokens.hip", "select.hip", "decode.hip", "step.hip", "prefill.hip",
           "probe.hip"]

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Wall", "-Wno-unused-function",
    "-Wno-pass-failed",   # large bitonic sorts keep their outer loops (no scratch)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # A single-lane atomic whose result is used later must not be rewritten
    # into a wave-wide one: that rewrite waits for the result (and every
    # load in flight) right after the atomic.
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    "-I", INCLUDE, "-I", CSRC,
]


def hipcc() -> str:
    h = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(h):
        raise RuntimeError("hipcc not found")
    return h


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [hipcc(), *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    # The host pass does not know the device-only feature name; drop that note.
    noise = "'-packed-fp32-ops' is not a recognized feature"
    msg = "\n".join(l for l in r.stderr.splitlines() if noise not in l).strip()
    if msg:
        print(msg, file=sys.stderr)
    return obj


def build_binding() -> str:
    """The marshalling module (see csrc/binding.cpp)."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc())))
    tmp = BINDING + f".tmp{os.getpid()}"
    cmd = [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-I", INCLUDE,
           "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(rocm, "include"),
           "-isystem", sysconfig.get_paths()["include"], "-Wall",
           f'-DSPOT_TORCH="{torch.__version__}"',
           os.path.join(CSRC, "binding.cpp"), "-o", tmp, "-L", os.path.join(root, "lib"),
           "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10", "-lc10_hip",
           f"-Wl,-rpath,{os.path.join(root, 'lib')}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for binding.cpp:\n{r.stderr}")
    os.replace(tmp, BINDING)
    return BINDING


def binding_fits() -> bool:
    """Whether a marshalling module is there and was built against this torch (whose
    tensor layout it relies on; another torch's may well import)."""
    import torch
    if not os.path.exists(BINDING):
        return False
    with open(BINDING, "rb") as f:
        return f"spot binding for torch {torch.__version__}\0".encode() in f.read()


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(min(len(SOURCES) + 1, os.cpu_count() or 4)) as ex:
        binding = ex.submit(build_binding)
        objs = list(ex.map(_compile, SOURCES))
        binding.result()
    tmp = SO + f".tmp{os.getpid()}"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, SO)
    if verbose:
        print(f"built {SO}")
    return SO


def stale() -> bool:
    if not os.path.exists(SO):
        return True
    t = min(os.path.getmtime(f) for f in (SO, BINDING) if os.path.exists(f))
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(INCLUDE, "spot.h")]
    return any(os.path.getmtime(p) > t for p in deps)


if __name__ == "__main__":
    build(verbose=True)
