"""The staged host copies against a stand-in for the HIP runtime (compiled and
run here): the device that is current on the caller's thread, the data of
copies both ways, and what becomes of errors."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# a runtime of two devices whose streams are small numbers, stream s on device s
RUNTIME = r"""
#pragma once
#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>
enum hipError_t { hipSuccess = 0, hipErrorInvalidResourceHandle = 400, hipErrorOutOfMemory = 2 };
enum hipMemoryType { hipMemoryTypeUnregistered = 0, hipMemoryTypeHost = 1 };
struct hipPointerAttribute_t { hipMemoryType type; };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost };
constexpr unsigned hipHostMallocDefault = 0, hipEventDisableTiming = 2;
struct Event { int device; };
using hipEvent_t = Event *;
using hipStream_t = std::intptr_t;
inline thread_local int g_current = 0;
inline std::atomic<int> g_copies{0}, g_pinned{0}, g_events{0};
inline std::atomic<int> g_fail_copy{-1};  // the copy that fails
inline hipError_t hipGetDevice(int *d) { *d = g_current; return hipSuccess; }
inline hipError_t hipSetDevice(int d) { g_current = d; return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline std::atomic<int> g_known{0};  // -1: the runtime has no answer
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) {
    a->type = g_known > 0 ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
    return g_known < 0 ? hipErrorInvalidResourceHandle : hipSuccess;
}
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned) { ++g_pinned; *p = malloc(n); return hipSuccess; }
inline hipError_t hipHostFree(void *p) { --g_pinned; free(p); return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { ++g_events; *e = new Event{g_current}; return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { --g_events; delete e; return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    return e->device == (int)s ? hipSuccess : hipErrorInvalidResourceHandle;
}
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    if (g_copies++ == g_fail_copy) return hipErrorInvalidResourceHandle;
    memcpy(d, s, n);
    return hipSuccess;
}
"""

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "lbfss_hostcopy.hpp"
int main(int argc, char **argv) {  // current device, down, bytes, the copy that fails, known
    g_current = atoi(argv[1]);
    const bool down = atoi(argv[2]);
    const size_t n = atol(argv[3]);
    g_fail_copy = atoi(argv[4]);
    g_known = atoi(argv[5]);
    std::vector<unsigned char> host(n), dev(n);
    for (size_t i = 0; i < n; ++i) (down ? dev : host)[i] = (unsigned char)(i * 2654435761u >> 24);
    hipError_t e;
    {
        lbfss::HostStage stage(1, 1);
        e = down ? stage.to_host(host.data(), dev.data(), n) : stage.to_device(dev.data(), host.data(), n);
    }
    printf("%d %d %d %d %d %d\n", (int)e, host == dev, g_current, g_pinned.load(), g_events.load(), g_copies.load());
}
"""


@pytest.fixture(scope="module")
def copy(tmp_path_factory):
    d = tmp_path_factory.mktemp("hostcopy")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", str(d), "-I",
                    os.path.join(ROOT, "paper_1202_4748_amd", "csrc"), "-o", str(d / "t"), str(d / "t.cpp")], check=True)

    def run(current, down, n, fail=-1, known=0):
        r = subprocess.run([str(d / "t"), str(current), str(int(down)), str(n), str(fail), str(known)],
                           capture_output=True, text=True, check=True, timeout=60)
        return tuple(map(int, r.stdout.split()))

    return run


@pytest.mark.parametrize("down", [False, True])
@pytest.mark.parametrize("n", [1000, 6 << 20, (6 << 20) - 8, (37 << 20) + 8])
@pytest.mark.parametrize("current", [0, 1])
def test_copies_with_any_device_current(copy, current, n, down):
    """No error, the data, the caller's device as it was, nothing left over."""
    assert copy(current, down, n)[:5] == (0, 1, current, 0, 0)


@pytest.mark.parametrize("down", [False, True])
@pytest.mark.parametrize("current", [0, 1])
def test_a_failed_piece_is_reported(copy, current, down):
    err, _, dev, pinned, events, _ = copy(current, down, 20 << 20, 5)
    assert (err, dev, pinned, events) == (400, current, 0, 0)


@pytest.mark.parametrize("down", [False, True])
def test_memory_the_runtime_knows_goes_in_one_copy(copy, down):
    """Pinned arrays of the caller are not passed through the pieces; memory
    that the runtime has no answer for is taken for ordinary memory."""
    assert copy(0, down, 20 << 20, known=1) == (0, 1, 0, 0, 0, 1)
    assert copy(0, down, 20 << 20, known=0) == copy(0, down, 20 << 20, known=-1) == (0, 1, 0, 0, 0, 20)
