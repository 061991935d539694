"""The host threads of large copies and scans (qmi_team.h), compiled by itself: every item is worked on
once, also where threads cannot be started, for want of memory as much as of threads (an exception
that leaves started threads behind would end the process)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1412_1840_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <new>
#include <system_error>
#include <vector>
#include "qmi_team.h"

static std::atomic<int> allowed{-1};  // allocations until one fails; -1: all succeed
void* operator new(std::size_t n) {
    int left = allowed.load();
    while (left > 0 && !allowed.compare_exchange_weak(left, left - 1)) {}
    if (left == 0) throw std::bad_alloc();
    if (void* p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main() {
    for (int fail = -1; fail < 8; ++fail)
        for (int n : {0, 1, 2, 7, 1000}) {
            std::vector<std::atomic<int>> seen(n);
            allowed = fail;
            qmi::run_team(n, [&](int64_t k) { seen[k].fetch_add(1); });
            allowed = -1;
            for (int k = 0; k < n; ++k)
                if (seen[k] != 1) return 1;
        }
    std::puts("ok");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_threads_that_cannot_be_started(tmp_path):
    src, exe = tmp_path / "team.cpp", tmp_path / "team"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, "-o", str(exe), str(src)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "ok\n", (out.returncode, out.stderr)
