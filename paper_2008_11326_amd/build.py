"""Build libgpp.so (HIP, gfx950 only) and _binding.so in-tree.

    python -m paper_2008_11326_amd.build        # or build() from Python
    python -m paper_2008_11326_amd.build --define GPP_FWD_COLS=1 --out $VDIR/libgpp_c1.so

The second form builds a variant with compile-time tuning knobs (the
GPP_* macros the sources document) into a library of its own, for
measurement; the package loads it when GPP_LIBRARY names it.

Each .hip source compiles to an object with hipcc for gfx950, then they
link into paper_2008_11326_amd/libgpp.so.  Packed-fp32 instructions are
disabled for all device code.  build() also compiles the native side of the
Python binding (host code against torch's headers) into _binding.so.
"""
import hashlib
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJDIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libgpp.so")
BINDING = os.path.join(PKG, "_binding.so")
BINDING_SOURCE = "gpp_binding.cpp"
SOURCES = ["gpp_api.hip", "gpp_fwd.hip", "gpp_bwd.hip", "gpp_batched.hip", "gpp_plan.hip",
           "gpp_ladder.hip", "gpp_noalloc.hip",
           "gpp_microbench.hip"]
HEADERS = ["gpp_device.h", "gpp_fwd_tile.h", "gpp_fwd_shape.h", "gpp_bwd_shape.h",
           "gpp_internal.h"]
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-fPIC", "-std=c++17",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result", f"-I{INCLUDE}", f"-I{CSRC}",
]
# The tile loops ask for the next group's values ahead of their
# arithmetic; with machine sinking on, the compiler moves those loads back
# behind a branch, right before their use.
EXTRA_FLAGS = {src: ["-mllvm", "-disable-machine-sink"]
               for src in ("gpp_fwd.hip", "gpp_batched.hip", "gpp_bwd.hip")}

# What the batched plan's tuning candidates are compiled from.
TUNED = ["gpp_batched.hip", "gpp_fwd_tile.h", "gpp_fwd_shape.h", "gpp_device.h", "gpp_internal.h",
         "gpp_plan.hip"]


def kernels_id(defines=()) -> str:
    """Names the kernels a tuned choice was timed with (gpp_plan.hip)."""
    h = hashlib.sha256(repr((FLAGS[:-2], sorted(EXTRA_FLAGS.items()), list(defines))).encode())
    for f in TUNED:
        with open(os.path.join(CSRC, f), "rb") as src:
            h.update(src.read())
    return h.hexdigest()[:8]


def _compile(src: str, verbose: bool, objdir: str = OBJDIR, defines=()) -> str:
    obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
    if src == "gpp_plan.hip":
        defines = [*defines, f'GPP_KERNELS_ID="{kernels_id(defines)}"']
    cmd = [HIPCC, *FLAGS, *EXTRA_FLAGS.get(src, []), *[f"-D{d}" for d in defines], "-c",
           os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass does not know the packed-fp32 feature; drop that note
    err = "\n".join(l for l in r.stderr.splitlines()
                    if "packed-fp32-ops" not in l and l.strip())
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err and verbose:
        print(err, file=sys.stderr)
    return obj


def build_binding(verbose: bool = False) -> str:
    """Compile the native side of the Python binding (csrc/gpp_binding.cpp)
    against the installed torch (always rebuilds)."""
    import torch
    root = torch.__path__[0]
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = BINDING + ".tmp"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-fPIC", "-shared", "-std=c++17", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-D__HIP_PLATFORM_AMD__=1", f"-I{INCLUDE}",
           *[f"-isystem{d}" for d in (os.path.join(root, "include"),
                                      os.path.join(root, "include/torch/csrc/api/include"),
                                      sysconfig.get_paths()["include"],
                                      os.path.join(rocm, "include"))],
           os.path.join(CSRC, BINDING_SOURCE), "-o", tmp, f"-L{root}/lib", "-lc10", "-lc10_hip",
           "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed for {BINDING_SOURCE}:\n{r.stderr}")
    os.replace(tmp, BINDING)
    return BINDING


def build(verbose: bool = False, defines=(), out: str = LIB) -> str:
    """Compile every HIP source for gfx950 and link libgpp.so (always
    rebuilds).  With defines (NAME=VALUE strings) the objects go to a
    directory of their own next to `out`, which must then be given too."""
    if defines and os.path.abspath(out) == LIB:
        raise ValueError("a variant build needs its own output path")
    objdir = OBJDIR if not defines else os.path.splitext(os.path.abspath(out))[0] + "_obj"
    os.makedirs(objdir, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        # a variant build shares the binding, which finds the library at run time
        binding = None if defines else ex.submit(build_binding, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose, objdir, defines), SOURCES))
        if binding:
            binding.result()
    tmp = out + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    return out


def is_stale() -> bool:
    if not (os.path.exists(LIB) and os.path.exists(BINDING)):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(BINDING))
    files = [os.path.join(CSRC, f) for f in SOURCES + HEADERS + [BINDING_SOURCE]]
    files += [os.path.join(INCLUDE, h) for h in os.listdir(INCLUDE)]
    return any(os.path.getmtime(f) > t for f in files)


if __name__ == "__main__":
    import argparse
    ap = argparse.ArgumentParser(description="build libgpp.so for gfx950")
    ap.add_argument("--define", action="append", default=[], metavar="NAME=VALUE")
    ap.add_argument("--out", default=LIB)
    a = ap.parse_args()
    build(verbose=True, defines=a.define, out=a.out)
