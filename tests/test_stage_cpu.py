"""Copies without page-locked memory (qmi_stage.h), compiled against a HIP whose queued copies run
when the stream is waited for, as they may on a device: the sources of an upload and the targets of
a download may go once the call returns, also with an error."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1412_1840_amd", "csrc")

HIP = r"""
#pragma once
#include <cstdlib>
#include <cstring>
#include <vector>
typedef int hipError_t;
typedef int hipStream_t;
typedef void* hipEvent_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost };
enum { hipHostMallocDefault = 0, hipEventDisableTiming = 2 };
struct Queued { void* dst; const void* src; size_t bytes; };
inline std::vector<Queued> queue;
inline bool fail_host_malloc = false;
inline int fail_copy = -1;  // copies until one cannot be queued
inline hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind, hipStream_t) {
    if (fail_copy >= 0 && fail_copy-- == 0) return hipErrorOutOfMemory;
    queue.push_back({dst, src, bytes});
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) {
    for (const Queued& q : queue) std::memcpy(q.dst, q.src, q.bytes);
    queue.clear();
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (fail_host_malloc) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    return hipSuccess;
}
inline hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = e; return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipStreamSynchronize(0); }
"""

PROGRAM = r"""
#include <cstdio>
#include <numeric>
#include "qmi_stage.h"

int main() {
    for (bool locked : {false, true})
        for (int fail : {-1, 1}) {
            qmi::Stage sg;
            std::vector<int> a(1000), b(3), dev(4096, -1);
            std::iota(a.begin(), a.end(), 1);
            b = {7, 8, 9};
            qmi::Upload up;
            const size_t at_a = up.add(a.data(), 4000), at_b = up.add(b.data(), 12);
            fail_host_malloc = !locked;
            fail_copy = locked && fail > 0 ? 0 : fail;
            const bool good = qmi::upload(sg, up, (char*)dev.data(), 0, 0, true) == hipSuccess;
            fail_copy = -1;
            if (good != (fail < 0)) return 1;
            std::fill(a.begin(), a.end(), 0);  // the caller's arrays are no longer its own
            std::fill(b.begin(), b.end(), 0);
            if (!locked && !queue.empty()) return 2;
            hipStreamSynchronize(0);
            if (good && (dev[at_a / 4] != 1 || dev[at_a / 4 + 999] != 1000 || dev[at_b / 4 + 2] != 9))
                return 3;
            if (!locked) {
                qmi::Download dn;
                dn.add(a.data(), dev.data() + at_a / 4, 4000);
                dn.add(b.data(), dev.data() + at_b / 4, 12);
                fail_copy = fail;
                if ((qmi::download(sg, dn, 0, true) == hipSuccess) != (fail < 0)) return 4;
                if (!queue.empty()) return 5;
                fail_copy = -1;
            }
            sg.release();
        }
    std::puts("ok");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_host_memory_may_go_after_a_copy(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    src, exe = tmp_path / "stage.cpp", tmp_path / "stage"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", str(tmp_path), "-I", CSRC,
                    "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "ok\n", (out.returncode, out.stderr)
