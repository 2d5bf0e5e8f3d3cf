"""Builds libfastgs_hip.so (gfx950) in-tree with hipcc, and _marshal (binding.py's native half, host code, for this Python and
this torch) with g++.
`python -m paper_2511_04283_amd.build`."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libfastgs_hip.so")
# (another Python looks for a file of another name; another torch would load this one: it says which it was built against)
MARSHAL_SRC, MARSHAL = os.path.join(CSRC, "marshal.cpp"), os.path.join(PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))


def marshal_stamp() -> str:
    import torch
    return f"built against torch {torch.__version__}"


HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",           # the fp32 operation order is part of the contract with the CPU oracle
    "-munsafe-fp-atomics",         # native global/LDS fp32 atomic add
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def is_stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(MARSHAL) or os.path.getmtime(MARSHAL_SRC) > os.path.getmtime(MARSHAL):
        return True
    with open(MARSHAL, "rb") as f:
        if marshal_stamp().encode() not in f.read():
            return True
    deps = sources() + glob.glob(os.path.join(CSRC, "*.hpp")) + [os.path.join(ROOT, "include", "fastgs.h")]
    return any(os.path.getmtime(d) > os.path.getmtime(LIB) for d in deps)


def source_digest() -> str:
    """Digest of the HIP sources (a measurement stored under profiles/ names the kernels it was made on with it)."""
    import hashlib
    h = hashlib.sha256()
    for f in sources() + sorted(glob.glob(os.path.join(CSRC, "*.hpp"))):
        h.update(open(f, "rb").read())
    return h.hexdigest()[:16]


def build(verbose: bool = False, extra=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", LIB, *sources()]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    build_marshal(verbose)
    return LIB


def build_marshal(verbose: bool = False) -> str:
    import torch
    from torch.utils import cpp_extension
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f'-DSTAMP="{marshal_stamp()}"', f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *(f"-I{d}" for d in [sysconfig.get_paths()["include"], *cpp_extension.include_paths()]), "-o", MARSHAL, MARSHAL_SRC,
           "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return MARSHAL


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
