"""Copies of results to the caller (host code), with a stand-in for the HIP
runtime: device memory is ordinary memory, and page-locked memory, streams and
events are counted. Every size where the way of copying changes, with and without
page-locked memory to be had."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2109_12565_amd", "csrc")
HIP = r"""
#pragma once
#include <cstdlib>
#include <cstring>
typedef int hipError_t;
typedef void* hipStream_t;
typedef void* hipEvent_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipHostMallocDefault = 0, hipMemcpyDeviceToHost = 2,
       hipEventDisableTiming = 2 };
struct Fake { int refuse, live, pinned, copies, last; };
inline Fake& fake() { static Fake f{}; return f; }
inline hipError_t hipGetLastError() { const int e = fake().last; fake().last = 0; return e; }
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (fake().refuse) { *p = (void*)1; return fake().last = hipErrorOutOfMemory; }
  ++fake().live; ++fake().pinned; *p = std::malloc(n); return hipSuccess;
}
inline hipError_t hipHostFree(void* p) { --fake().live; std::free(p); return hipSuccess; }
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int, hipStream_t) {
  ++fake().copies; std::memcpy(d, s, n); return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = std::malloc(1); return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
"""
SOURCE = r"""
#include "readout.hpp"
extern "C" {
void* make() { return new tlbh::Readout; }
void drop(void* r) { delete static_cast<tlbh::Readout*>(r); }
void* page(void* r) { return static_cast<tlbh::Readout*>(r)->page(); }
int fetch(void* r, const void* src, size_t bytes, int parts, void** dst) {
  return static_cast<tlbh::Readout*>(r)->fetch(src, bytes, parts, dst, nullptr);
}
int* counts() { return &fake().refuse; }
}
"""
MIB = 1 << 20


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("readout")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(HIP)
    (d / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-pthread", "-I", str(d), "-I", CSRC,
                    str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    lib = ctypes.CDLL(str(d / "t.so"))
    lib.make.restype = lib.page.restype = ctypes.c_void_p
    lib.counts.restype = ctypes.POINTER(ctypes.c_int)
    lib.drop.argtypes = lib.page.argtypes = [ctypes.c_void_p]
    lib.fetch.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_void_p]
    return lib


@pytest.fixture
def reader(lib):
    c = lib.counts()
    for k in range(5):
        c[k] = 0
    r = lib.make()
    yield lib, r, c
    if r:
        lib.drop(r)


def fetch(lib, r, nbytes, parts, leave_out=(), shift=0):
    """Copy, check every byte and the bytes around, return the status."""
    rng = np.random.default_rng(nbytes + parts)
    src = rng.integers(0, 255, nbytes * parts, dtype=np.uint8)
    room = [np.full(nbytes + 64, 255, np.uint8) for _ in range(parts)]
    dst = (ctypes.c_void_p * parts)(*(None if k in leave_out else room[k].ctypes.data + 8 + shift
                                      for k in range(parts)))
    rc = lib.fetch(r, src.ctypes.data, nbytes, parts, dst)
    for k in range(parts):
        inner = room[k][8 + shift:8 + shift + nbytes]
        if k in leave_out:
            assert (room[k] == 255).all()
        elif rc == 0:
            assert np.array_equal(inner, src[k * nbytes:(k + 1) * nbytes]), k
            assert (room[k][:8 + shift] == 255).all() and (room[k][8 + shift + nbytes:] == 255).all()
    return rc


SIZES = [(8, 5), (6554 * 2, 5), (13108, 5), (65536, 1), (65537, 1), (2 * MIB, 1), (2 * MIB // 5, 5),
         (2 * MIB // 5 + 8, 5), (7 * MIB, 5), (32 * MIB - 8, 1), (32 * MIB, 1), (48 * MIB // 5 + 8, 5),
         (16 * MIB + 40, 3), (33 * MIB + 1, 2)]


@pytest.mark.parametrize("refuse", [0, 1])
@pytest.mark.parametrize("nbytes,parts", SIZES)
def test_blocks_arrive_with_and_without_page_locked_memory(reader, nbytes, parts, refuse):
    lib, r, c = reader
    c[0] = refuse
    assert fetch(lib, r, nbytes, parts, shift=nbytes % 3) == 0
    assert c[4] == 0            # no error is left for the next check
    if parts > 2:
        assert fetch(lib, r, nbytes, parts, leave_out=(1,)) == 0
    if refuse:
        assert not lib.page(r) and c[2] == 0 and c[4] == 0
        c[0] = 0                # and once there is some again
        assert lib.page(r) and fetch(lib, r, nbytes, parts) == 0


def test_small_read_outs_allocate_once(reader):
    """Whatever the order, one page and one ring, which grows once for large
    blocks; a single small block takes neither."""
    lib, r, c = reader
    assert lib.page(r) and c[2] == 1
    assert fetch(lib, r, 512 * 1024, 1) == 0 and c[2] == 1
    for nbytes, parts in ((64, 5), (512, 2), (65536, 2), (2 * MIB // 5, 5), (100000, 5), (65536, 5), (512 * 1024, 1)):
        assert fetch(lib, r, nbytes, parts) == 0
    assert c[2] == 2 and c[1] == 2
    for _ in range(2):
        assert fetch(lib, r, 33 * MIB, 2) == 0
        assert fetch(lib, r, 100000, 5) == 0
    assert c[2] == 3 and c[1] == 2
