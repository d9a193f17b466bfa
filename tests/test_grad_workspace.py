"""The gradient's workspace (csrc/grad_workspace.hpp, built for the host with a counting allocator):
allocated on first use and kept, also where only a workspace for chunks of samples could be had."""
import ctypes
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2411_03289_amd", "csrc")


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    out = str(tmp_path_factory.mktemp("ws") / "libws.so")
    subprocess.run([cxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC,
                    os.path.join(HERE, "grad_workspace_check.cpp"), "-o", out], check=True, capture_output=True)
    lib = ctypes.CDLL(out)
    size = ctypes.c_size_t
    lib.ws_new.restype, lib.ws_new.argtypes = ctypes.c_void_p, [size, size, size]
    lib.ws_call.argtypes = lib.ws_capacity.argtypes = [ctypes.c_void_p, size]
    lib.ws_bytes.restype = size
    for f in ("ws_delete", "ws_allocs", "ws_frees", "ws_bytes"):
        getattr(lib, f).argtypes = [ctypes.c_void_p]
    return lib


def test_enough_memory_is_asked_for_once(L):
    s = L.ws_new(10_000, 100, 1000)
    assert [L.ws_call(s, 700) for _ in range(3)] == [1, 1, 1]
    assert (L.ws_allocs(s), L.ws_frees(s), L.ws_bytes(s)) == (1, 0, 1100)
    L.ws_delete(s)


@pytest.mark.parametrize("limit,chunks", [(700, 2), (600, 2), (500, 3), (200, 10)])
def test_a_workspace_for_chunks_is_kept(L, limit, chunks):
    s = L.ws_new(1099, 100, 1000)   # one byte short of the whole
    assert L.ws_call(s, limit) == chunks
    assert (L.ws_allocs(s), L.ws_frees(s)) == (2, 0)
    held = L.ws_bytes(s)
    L.ws_capacity(s, 0)             # other code took the rest
    for other in (limit, limit + 300, 150, limit):   # whatever the call's own limit
        assert L.ws_call(s, other) == chunks
    assert (L.ws_allocs(s), L.ws_frees(s), L.ws_bytes(s)) == (2, 0, held)
    L.ws_delete(s)


def test_no_memory_is_reported_and_asked_for_again(L):
    s = L.ws_new(300, 100, 1000)
    assert L.ws_call(s, 700) == 0
    assert (L.ws_allocs(s), L.ws_bytes(s)) == (2, 0)
    L.ws_capacity(s, 2000)
    assert L.ws_call(s, 700) == 1
    L.ws_delete(s)


def test_nothing_smaller_is_tried_within_the_limit(L):
    s = L.ws_new(300, 100, 1000)
    assert L.ws_call(s, 1100) == 0
    assert L.ws_allocs(s) == 1
    L.ws_delete(s)
