"""Build libsar_mi355x.so (the product), _binding.so (the Python side of its hot calls) and libsar_bench.so
(bench.py's bandwidth probes) from csrc/ with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsar_mi355x.so")
SOURCES = ["builder.hip", "spmm.hip", "gat.hip", "gat_slices.hip", "gat_joint_f32.hip", "gat_joint_bf16.hip", "linear.hip",
           "linear_split.hip", "linear_few.hip"]
BENCH_LIB = os.path.join(HERE, "libsar_bench.so")
BENCH_SOURCES = ["probe.hip"]
BINDING = os.path.join(HERE, "_binding.so")
BINDING_SOURCE = "binding.cpp"

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-munsafe-fp-atomics",
    # packed fp32 VALU forms are kept off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def binding_for() -> str:
    """The interpreter and the torch whose objects the binding reads by their headers' layout."""
    import torch
    return "python %d.%d, torch %s %s" % (*sys.version_info[:2], torch.__version__, torch.version.git_version)


def binding_flags():
    """The binding is host code that reads torch's tensors: compiled against the installed torch's headers."""
    from torch.utils import cpp_extension
    return ["-O2", '-DSAR_BUILT_FOR="%s"' % binding_for(), "-std=c++17", "-fPIC", "-w", "-DUSE_ROCM", "-isystem", sysconfig.get_paths()["include"],
            *[f for path in cpp_extension.include_paths() for f in ("-isystem", path)]]


def binding_link_flags():
    """Linked against the library beside it; torch's own are loaded by the time it is imported."""
    from torch.utils import cpp_extension
    return ["-L" + HERE, "-lsar_mi355x", "-Wl,-rpath,$ORIGIN",
            *["-L" + path for path in cpp_extension.library_paths()], "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared library in-tree.  Always rebuilds."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src: str) -> str:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        flags = binding_flags() if src == BINDING_SOURCE else HIPCC_FLAGS
        cmd = [hipcc, *flags, "-c", os.path.join(CSRC, src), "-o", obj]
        res = subprocess.run(cmd, capture_output=True, text=True)
        noise = "packed-fp32-ops"
        err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    def link(objs, lib, flags=()):
        tmp = lib + ".%d.tmp" % os.getpid()
        res = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs, *flags],
                             capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("link failed:\n" + res.stderr)
        os.replace(tmp, lib)

    # (the libraries know nothing of torch: they are built where the binding cannot be, too)
    with ThreadPoolExecutor(max_workers=8) as pool:
        binding = pool.submit(compile_one, BINDING_SOURCE)
        objs = list(pool.map(compile_one, SOURCES + BENCH_SOURCES))
    link(objs[:len(SOURCES)], LIB)
    link(objs[len(SOURCES):], BENCH_LIB)
    link([binding.result()], BINDING, binding_link_flags())
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
