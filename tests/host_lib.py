"""The library's runtime (csrc/ee_api.hip) built for the CPU over
tests/host_runtime.cpp, behind the binding's own Engine."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

from tests.conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2609_14144_amd", "csrc")
HIP_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


def build_host_lib(out_dir):
    gxx = shutil.which("g++")
    if not gxx or not os.path.exists(os.path.join(HIP_INCLUDE, "hip", "hip_runtime.h")):
        pytest.skip("no g++ or no HIP headers")
    out = os.path.join(str(out_dir), "libee_host.so")
    # -Bsymbolic: the stand-ins are used even where a HIP runtime is loaded
    subprocess.run([gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                    "-I", HIP_INCLUDE, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    "-x", "c++", os.path.join(CSRC, "ee_api.hip"), os.path.join(ROOT, "tests", "host_runtime.cpp"),
                    "-o", out], check=True)
    return out


@pytest.fixture(scope="session")
def host_lib(tmp_path_factory):
    """(binding module with its library replaced, the library)."""
    B = pytest.importorskip("paper_2609_14144_amd._binding", exc_type=ImportError)
    path = build_host_lib(tmp_path_factory.mktemp("host"))
    real, real_path = B.lib, B.lib_path
    B.lib_path = path
    try:
        lib = B._load()
    finally:
        B.lib_path = real_path
    lib.host_device_limit.argtypes = [C.c_uint64]
    lib.host_device_bytes.restype = C.c_uint64
    return lib


@pytest.fixture
def host(host_lib, monkeypatch):
    """The host library in the place of libee.so for one test, which must not
    hand the device a range outside its buffers."""
    from paper_2609_14144_amd import _binding as B
    monkeypatch.setattr(B, "lib", host_lib)
    bad = host_lib.host_bad_ranges()
    yield host_lib
    host_lib.host_fail_alloc(0, 0)
    host_lib.host_fail_alloc(1, 0)
    host_lib.host_device_limit(2 ** 64 - 1)
    host_lib.host_max_wgs(1)
    assert host_lib.host_bad_ranges() == bad, "a launch was handed memory outside its buffers"
