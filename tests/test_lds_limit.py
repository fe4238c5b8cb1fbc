"""Host logic of the kernels' dynamic LDS limit (lds_limit.h), compiled with g++
at test time against stand-ins of the HIP calls: once per device and size, never
lowered, and a failure is not remembered."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = tmp_path_factory.mktemp("lds") / "liblds_limit.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread", "-Wall", "-Werror",
                    "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include",
                    f"-I{os.path.join(ROOT, 'paper_2405_19056_amd', 'csrc')}", "-Wl,-Bsymbolic",
                    os.path.join(ROOT, "tests", "native", "lds_limit_harness.cpp"),
                    "-o", str(out)], check=True)
    L = ctypes.CDLL(str(out))
    L.l_create.restype = ctypes.c_void_p
    L.l_destroy.argtypes = [ctypes.c_void_p]
    L.l_raise.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return L


def test_limit_is_raised_per_device_and_not_after_a_failure(lib):
    p = lib.l_create()
    at = lib.l_calls()

    def calls(device, bytes_, fail=0, want=0):
        nonlocal at
        assert lib.l_raise(p, device, fail, bytes_) == want
        n, at = lib.l_calls() - at, lib.l_calls()
        return n
    assert calls(0, 100000) == 1 and lib.l_last() == 100000
    assert calls(0, 100000) == 0
    assert calls(0, 70000) == 0                      # not lowered
    assert calls(0, 150000) == 1 and lib.l_last() == 150000
    assert calls(1, 100000) == 1                     # another device
    assert calls(2, 100000, fail=1, want=-1) == 1
    assert calls(2, 100000) == 1                     # tried again
    assert calls(2, 100000) == 0
    assert calls(99, 1000) == 1 and calls(99, 1000) == 1   # past the record: every time
    lib.l_destroy(p)
