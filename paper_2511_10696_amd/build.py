"""Build libpi_attn.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2511_10696_amd.build          # or build() from Python

Each ``csrc/*.hip`` is compiled to an object under ``_build/`` (in parallel)
and linked into ``paper_2511_10696_amd/libpi_attn.so``; ``csrc/binding.cpp``,
the native marshalling of torch tensors, becomes
``paper_2511_10696_amd/_binding.so`` beside it.  The library needs neither
torch nor Python's headers; where they are missing it is built alone, and the
Python code marshals every call.
"""
from __future__ import annotations

import glob
import importlib.util
import os
import re
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB_PATH = os.path.join(PKG, "libpi_attn.so")
BINDING_PATH = os.path.join(PKG, "_binding.so")
ARCH = "gfx950"

# Packed-FP32 VALU instructions are disabled for every kernel (hipcc would
# otherwise form them from float2-style code).  MFMA accumulators are kept in
# ordinary VGPRs (the softmax rescales them with VALU instructions; the AGPR
# form would copy them back and forth).
DEVICE_FLAGS = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
VGPR_FORM = ["-mllvm", "-amdgpu-mfma-vgpr-form"]
COMMON = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall",
          "-I", os.path.join(ROOT, "include")] + DEVICE_FLAGS


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    path = os.path.join(rocm, "bin", "hipcc")
    return path if os.path.exists(path) else "hipcc"


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


# The compiler's per-kernel resource remarks; the build fails if any kernel
# needs private (scratch) memory, i.e. spills registers.
RESOURCE_REMARKS = ["-Rpass-analysis=kernel-resource-usage"]


def scratch_users(remarks: str) -> list[str]:
    """Kernels whose resource remark reports a nonzero ScratchSize."""
    users, name = [], None
    for line in remarks.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            continue
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and int(m.group(1)) > 0:
            users.append(f"{name} ({m.group(1)} bytes/lane)")
    return users


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    cmd = [hipcc(), *COMMON, *VGPR_FORM, *RESOURCE_REMARKS, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    spills = scratch_users(r.stderr)
    if spills:
        raise RuntimeError(f"{src}: kernels use scratch memory (register spills): " + ", ".join(spills))
    return obj


def _torch_init() -> str | None:
    """torch/__init__.py, if the binding can be built here: its C++ API and
    Python's headers are there."""
    spec = importlib.util.find_spec("torch")
    if spec is None or spec.origin is None:
        return None
    needed = [os.path.join(os.path.dirname(spec.origin), "include", "torch", "csrc", "Exceptions.h"),
              os.path.join(sysconfig.get_paths()["include"], "Python.h")]
    return spec.origin if all(map(os.path.exists, needed)) else None


def _build_binding(torch_init: str) -> None:
    """_binding.so: host code against torch's C++ API and libpi_attn.so."""
    tdir = os.path.dirname(torch_init)
    includes = [os.path.join(tdir, "include"), os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
                sysconfig.get_paths()["include"], os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")]
    tmp = BINDING_PATH + ".tmp"
    cmd = [hipcc(), "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-I", os.path.join(ROOT, "include")]
    for d in includes:
        cmd += ["-isystem", d]
    cmd += ["-shared", os.path.join(CSRC, "binding.cpp"), "-o", tmp, f"-L{PKG}", "-l:libpi_attn.so",
            "-Wl,-rpath,$ORIGIN", f"-L{os.path.join(tdir, 'lib')}"]
    cmd += [f"-l{x}" for x in ("c10", "c10_hip", "torch", "torch_cpu", "torch_python")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for binding.cpp:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, BINDING_PATH)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB_PATH + ".tmp"
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB_PATH)
    torch_init = _torch_init()
    if torch_init:
        _build_binding(torch_init)
    elif os.path.exists(BINDING_PATH):   # of another library
        os.remove(BINDING_PATH)
    if verbose:
        print(f"built {LIB_PATH}" + (f" and {BINDING_PATH}" if torch_init else
                                     "; no torch or Python headers: without the native marshalling"))
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
