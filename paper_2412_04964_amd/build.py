"""Compile the HIP sources for gfx950 into ``libfc.so`` and the torch binding into ``_fc_torch.so`` next to this file.

    python -m paper_2412_04964_amd.build

hipcc cross-compiles without a GPU.  Flags that matter for bit-parity with the
arithmetic contract in include/fc.h:
  -ffp-contract=off          no implicit fused multiply-add (fmaf is explicit)
  no fast-math, IEEE divide  hipcc defaults, left alone
  packed-fp32 ops disabled   the build never emits v_pk_*_f32
and one that matters for speed:
  -amdgpu-kernarg-preload-count=16   the leading kernel arguments arrive in scalar registers when a
                             wavefront starts instead of being read from memory first (gfx940 and
                             later); the kernels' wavefronts live for one tile, so the saved read
                             is 1 % of the fused kernel's time
"""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfc.so")
BENCH_LIB = os.path.join(HERE, "libfc_bench.so")      # measurement aid (include/fc_bench.h), not the product
# the product library with the kernels that use landing zones (the fused kernels, the one-launch all-reduce) compiled
# with -DFC_PLAIN_LANDING_READS (plain, compiler-ordered reads of the landing zones instead of the hand-ordered
# ones): the GPU tests run those cases through both
PLAIN_LIB = os.path.join(HERE, "libfc_plainreads.so")
# CPython extension between torch tensors and the C ABI (host code only; built against the installed torch)
TORCH_EXT = os.path.join(HERE, "_fc_torch.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    "--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
    "-I", INCLUDE, "-I", CSRC,
]

# (source, object suffix, extra defines)
UNITS = [("fc_api.hip", "api", []), ("fc_codec.hip", "codec", []), ("fc_wide.hip", "wide", []),
         ("fc_rot.hip", "rot", []), ("fc_rot_rows.hip", "rot_rows", []), ("fc_rot_fine.hip", "rot_fine", []), ("fc_rot_sim.hip", "rot_sim", []),
         ("fc_small.hip", "small", [])]
for _c in range(4):      # one unit per quantizer: asymmetric, symmetric, FP8, asymmetric with binary16 metadata
    UNITS.append(("fc_sim.hip", "sim_%d" % _c, ["-DFC_SIM_CODEC=%d" % _c]))
    UNITS.append(("fc_sim_wide.hip", "sim_wide_%d" % _c, ["-DFC_SIM_CODEC=%d" % _c]))
BENCH_UNITS = [("fc_bench.hip", "bench", [])]
for _bi in (4, 8):
    for _bo in (4, 8):
        UNITS.append(("fc_fused.hip", "fused_%d_%d" % (_bi, _bo),
                      ["-DFC_BITS_IN=%d" % _bi, "-DFC_BITS_OUT=%d" % _bo]))


LANDING_SOURCES = ("fc_fused.hip", "fc_sim.hip")
PLAIN_UNITS = [(src, tag + "_plain", defs + ["-DFC_PLAIN_LANDING_READS"]) for src, tag, defs in UNITS
               if src in LANDING_SOURCES]


def _compile(unit):
    src, tag, defs = unit
    obj = os.path.join(OBJDIR, tag + ".o")
    cmd = [HIPCC, *FLAGS, *defs, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (tag, " ".join(cmd), r.stderr))
    warn = [l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip()]
    return obj, "\n".join(warn)


def _compile_torch_ext():
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    tmp = TORCH_EXT + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-DFC_TORCH_VERSION=\"%s\"" % torch.__version__, "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           "-I", INCLUDE]
    for path in [*cpp_extension.include_paths(), sysconfig.get_paths()["include"],
                 os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include")]:
        cmd += ["-isystem", path]
    cmd += [os.path.join(CSRC, "fc_torch.cpp"), "-o", tmp]
    for path in cpp_extension.library_paths():
        cmd += ["-L" + path, "-Wl,-rpath," + path]
    cmd += ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compiling fc_torch.cpp failed:\n%s\n%s" % (" ".join(cmd), r.stderr))
    os.replace(tmp, TORCH_EXT)
    return r.stderr


def build(verbose: bool = False, jobs: int | None = None) -> str:
    """Compile every unit (always; this is the "does it build" check) and link.  The libraries need hipcc alone; without
    torch only the torch binding is left out."""
    os.makedirs(OBJDIR, exist_ok=True)
    jobs = jobs or min(8, os.cpu_count() or 1)
    with ThreadPoolExecutor(jobs) as ex:
        ext = ex.submit(_compile_torch_ext) if importlib.util.find_spec("torch") else None
        results = list(ex.map(_compile, UNITS + BENCH_UNITS + PLAIN_UNITS))
    objs = [o for o, _ in results]
    n_u, n_b = len(UNITS), len(BENCH_UNITS)
    shared = [o for o, (src, _, _) in zip(objs[:n_u], UNITS) if src not in LANDING_SOURCES]
    for lib, members in ((LIB, objs[:n_u]), (BENCH_LIB, objs[n_u:n_u + n_b]), (PLAIN_LIB, shared + objs[n_u + n_b:])):
        tmp = lib + ".tmp.%d" % os.getpid()
        cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp, *members]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n%s" % r.stderr)
        os.replace(tmp, lib)
    warnings = [w for _, w in results]
    warnings.append(ext.result() if ext else "torch is not installed: %s not built" % os.path.basename(TORCH_EXT))
    if verbose:
        for w in warnings:
            if w:
                print(w, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
