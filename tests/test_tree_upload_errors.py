"""Uploads of the tree's changes when a call of the runtime fails, on a device made of host memory (tree_on_fake_device.cpp)."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "tree_on_fake_device.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include",
                           os.path.join(HERE, "tree_on_fake_device.cpp"), "-o", so])
    lib = C.CDLL(so)
    lib.pa_tree_create.argtypes = [C.POINTER(C.c_void_p)]
    lib.pa_tree_insert.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int32, C.POINTER(C.c_int32)]
    lib.pa_tree_upload.argtypes = [C.c_void_p, C.c_void_p]
    lib.pa_tree_upload_stats.argtypes = [C.c_void_p] + [C.POINTER(C.c_int64)] * 3
    lib.pa_tree_destroy.argtypes = [C.c_void_p]
    lib.fake_check.argtypes = [C.c_void_p]
    lib.fake_fail.argtypes = [C.c_char_p, C.c_int]
    return lib


# After `at` uploads of changes one fails, three times: in the calls that every such upload makes, in those that it makes once its
# buffer has to grow, and in those of the first use of a buffer.
@pytest.mark.parametrize("at", [0, 1, 2])
@pytest.mark.parametrize("long_run", [False, True])
@pytest.mark.parametrize("call", ["hipHostMalloc", "hipHostGetDevicePointer", "hipEventCreateWithFlags", "hipEventSynchronize",
                                  "hipMemcpyAsync", "launch", "hipEventRecord"])
def test_an_upload_after_a_failed_one_is_whole(lib, call, long_run, at):
    rng = np.random.default_rng(at)
    tree, slot = C.c_void_p(), 0
    assert lib.pa_tree_create(C.byref(tree)) == 0

    def insert(n):
        nonlocal slot
        toks = rng.integers(0, 1000, n).astype(np.int32)
        toks[0] = 2000 + slot
        slots = np.arange(slot, slot + n, dtype=np.int32)
        slot += n
        assert lib.pa_tree_insert(tree, toks.ctypes.data, slots.ctypes.data, n, C.byref(C.c_int32())) == 0

    lib.fake_fail(b"", 0)
    insert(400000)
    assert lib.pa_tree_upload(tree, None) == 0
    for _ in range(at):
        insert(300)
        assert lib.pa_tree_upload(tree, None) == 0
    assert lib.fake_check(tree) == 0
    for _ in range(3):
        for n in ([20000, 500] if long_run else [500, 300]):
            insert(n)
        lib.fake_fail(call.encode(), 0)
        rc = lib.pa_tree_upload(tree, None)
        lib.fake_fail(b"", 0)
        if rc == 0:                          # (this upload makes no such call)
            assert lib.fake_check(tree) == 0
        for _ in range(3):                   # both transfer buffers again, and commands still queued while the next is made
            insert(30 if not long_run else 18000)
            assert lib.pa_tree_upload(tree, None) == 0
        assert lib.fake_check(tree) == 0
    full, part, last = C.c_int64(), C.c_int64(), C.c_int64()
    lib.pa_tree_upload_stats(tree, C.byref(full), C.byref(part), C.byref(last))
    assert part.value >= at + 6
    lib.pa_tree_destroy(tree)
