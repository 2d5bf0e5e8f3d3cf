"""Launches that a size could make larger than the GPU takes, from binsort.hip's host code on the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def launchers(tmp_path_factory):
    if not os.path.exists(HIPCC) or not shutil.which("objcopy"):
        pytest.skip("no hipcc / objcopy")
    out = str(tmp_path_factory.mktemp("launches"))
    csrc = os.path.join(ROOT, "paper_2511_04283_amd", "csrc")
    flags = ["-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-w", "-I", csrc, "-I",
             os.path.join(ROOT, "include")]
    for name, src in (("binsort", os.path.join(csrc, "binsort.hip")), ("stub", os.path.join(ROOT, "tests", "host_launch_stub.cpp"))):
        subprocess.run([HIPCC, *flags, "-c", src, "-o", f"{out}/{name}.o"], check=True)
    subprocess.run(["objcopy", "--wildcard", "--weaken-symbol=__hip_fatbin*", f"{out}/binsort.o"], check=True)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-o", f"{out}/libstub.so", f"{out}/binsort.o", f"{out}/stub.o"], check=True)
    return ctypes.CDLL(f"{out}/libstub.so")


@pytest.mark.parametrize("count", [1, 3, 1000, 12 * 358_000_000, 12 * (2 ** 31 - 1)])
def test_any_number_of_records_can_be_cleared(launchers, count):
    """A dense backward pass with the Compact Box clears twelve words for each of up to 2^31 candidate tiles; HIP refuses a launch of 2^32
    threads or more in one dimension."""
    fill = launchers._ZN2fs15launch_fill_u32EP12ihipStream_tPjjl
    fill.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_int64]
    assert fill(None, 4096, 0, count) == 0
    blocks, threads = (ctypes.c_longlong.in_dll(launchers, k).value for k in ("stub_blocks", "stub_threads"))
    assert 0 < blocks * threads < 2 ** 32
