"""Builds libtpo.so (the C-ABI library of the operator), libtpo_bench.so (the benchmark's
measurement aid) for gfx950 with hipcc and _tpo_torch.so (the native form of the binding's tensor
functions, host code), in-tree.

    python -m paper_2604_19906_amd.build          # compile every source and link

Every translation unit under ``csrc/`` is compiled to an object under ``_build/`` (in
parallel).  Those named ``bench_*`` are linked into ``paper_2604_19906_amd/libtpo_bench.so``
(``include/tpo_bench.h``), ``torch_binding.cpp`` against torch's libraries into
``paper_2604_19906_amd/_tpo_torch.so``, all others into ``paper_2604_19906_amd/libtpo.so``
(``include/tpo.h``).  hipcc cross-compiles for gfx950 without a GPU being present.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libtpo.so")
BENCH_LIB = os.path.join(HERE, "libtpo_bench.so")
TORCH_BINDING = os.path.join(HERE, "_tpo_torch.so")

ARCH = "gfx950"
# Packed-FP32 VALU instructions are switched off for all device code.
HIP_FLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wextra",
             "-Wno-unused-parameter",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             # keep MFMA accumulators in ordinary VGPRs (no AGPR copies around every tile)
             "-mllvm", "-amdgpu-mfma-vgpr-form",
             # the first 14 words of a kernel's arguments (the most there is room for) arrive in scalar
             # registers with the launch: a wavefront asks for its first words of u without waiting for a
             # scalar load.  Geometric means over all n, with / without: 1 .. 30 MB 0.96 .. 0.98 (operator,
             # separable form, halves, convection term), 100 MB 0.97 .. 0.99, 1 GB 0.99 .. 1.00
             # (a launch gets 0.12 us longer by it: settings that lose have their arguments held back, kHeld in
             # tpo_batch_rows.hpp)
             "-mllvm", "-amdgpu-kernarg-preload-count=14",
             "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")) and not f.startswith("torch_"))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    path = os.path.join(CSRC, src)
    cmd = ["hipcc"] + HIP_FLAGS + (["-x", "hip"] if src.endswith(".cpp") else []) + ["-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines()
                    if "is not a recognized feature for this target" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _build_torch_binding() -> None:
    import torch

    from .tpo import binding_versions

    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    include = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
               os.path.join(rocm, "include"), sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    tmp = TORCH_BINDING + f".tmp{os.getpid()}"
    cmd = (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f'-DTPO_BUILT_FOR="{binding_versions()}"']
           + ["-isystem" + d for d in include]
           + [os.path.join(CSRC, "torch_binding.cpp"), "-o", tmp, "-L" + os.path.join(root, "lib"),
              "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"])
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on torch_binding.cpp:\n" + r.stderr)
    os.replace(tmp, TORCH_BINDING)


def build(jobs: int = 8, verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max_workers=max(1, min(jobs, len(srcs) + 1))) as ex:
        binding = ex.submit(_build_torch_binding)
        objs = list(ex.map(_compile, srcs))
    for lib, part in ((LIB, [o for s_, o in zip(srcs, objs) if not s_.startswith("bench_")]),
                      (BENCH_LIB, [o for s_, o in zip(srcs, objs) if s_.startswith("bench_")])):
        tmp = lib + f".tmp{os.getpid()}"
        cmd = ["hipcc", "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp] + part
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n" + r.stderr)
        os.replace(tmp, lib)
        if verbose:
            print(f"built {lib} from {len(part)} sources")
    # The C libraries need hipcc alone.  Without torch, g++ or Python's headers the tensor functions keep their Python form; one left
    # from an earlier build does not stay.
    try:
        binding.result()
    except (ImportError, OSError, RuntimeError) as e:
        if os.path.exists(TORCH_BINDING):
            os.remove(TORCH_BINDING)
        warnings.warn(f"{TORCH_BINDING} is not built, tensor functions run in their Python form: {e}")
    else:
        if verbose:
            print(f"built {TORCH_BINDING}")
    return LIB


if __name__ == "__main__":
    build()
