"""The library's host code where a kernel launch fails: run against a HIP runtime without a device
(native/hip_stub.cpp), in a process of its own that loads nothing else of HIP.  Nothing here needs a GPU."""
import os
import subprocess
import sys

import pytest

import paper_2511_07421_amd as a3

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = r"""
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
L = C.CDLL(sys.argv[2])
maps = open("/proc/self/maps").read()
assert maps.count("libamdhip64") and "/opt/rocm" not in maps, "the stub must be the only HIP runtime here"
stub.stub_launches.restype = C.c_char_p
L.a3_sample_blocks.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int32, C.c_int64, C.c_void_p, C.c_int64,
                               C.c_void_p, C.c_int32, C.c_void_p, C.c_uint32, C.c_uint64, C.c_void_p]
L.a3_destroy.argtypes = [C.c_void_p]
A3_STATIC_MAP, STATIC = 512, sys.argv[3] == "static"
fan = (C.c_int32 * 2)(4, 3)
ctx = C.c_void_p()
assert L.a3_create(C.byref(ctx), 0, None, C.c_int64(8), 2, fan, A3_STATIC_MAP if STATIC else 0) == 0
mem = C.create_string_buffer(4096)   # stands for every device array: no kernel runs
maps = [C.addressof(mem), C.addressof(mem) + 2048]

def call(which, fail=b""):
    stub.stub_launches()
    stub.stub_fail_next(fail)
    rc = L.a3_sample_blocks(ctx, mem, mem, 4, 100, mem, 8, fan, 2, maps[which], 4 * 65536, 0, C.create_string_buffer(4096))
    made = b"k_cached_bits" in stub.stub_launches()
    stub.stub_fail_next(b"")
    return rc, made

# made once and kept; made by every call without the flag
assert call(0) == (0, True) and call(0) == (0, not STATIC)
for kernel in (b"k_frontier", b"k_cached_bits", b"k_sample", b"k_relabel"):
    # a call with another map fails on the way: neither map's classes and bitmap may be taken as there
    rc, _ = call(1, kernel)
    assert rc == -3, (kernel, rc)
    assert call(1) == (0, True), kernel
    assert call(1) == (0, not STATIC), kernel
    assert call(0, kernel)[0] == -3
    assert call(1) == (0, True), kernel
    assert call(0) == (0, True) and call(0) == (0, not STATIC), kernel
assert L.a3_destroy(ctx) == 0
print("ok")
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "libamdhip64.so.7")
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-shared", "-fPIC", "-Wall",
                    "-Wl,-soname,libamdhip64.so.7", "-Wl,--version-script=" + os.path.join(HERE, "native", "hip_stub.map"),
                    os.path.join(HERE, "native", "hip_stub.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("flag", ["static", "plain"])
def test_a_failed_launch_leaves_no_kept_map_behind(stub, flag):
    """A3_STATIC_MAP: what a context keeps of a device map is valid only once the whole call that makes it is queued"""
    a3.lib()
    res = subprocess.run([sys.executable, "-c", CHILD, stub, a3.library_path(), flag], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr
