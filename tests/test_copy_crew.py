"""The host threads of od_read (CopyCrew) where memory or threads run short:
every allocation of a read fails once, in turn, and the read either throws
std::bad_alloc or copies every byte; it never ends the process.  Host-only:
the class is compiled here with a counting allocator."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_12734_amd", "csrc")

PROGRAM = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>
#include "copy_crew.hpp"

static std::atomic<long> left{-1};   // allocations until one fails; -1: none does
void* operator new(size_t n) {
    if (left >= 0 && left-- == 0) throw std::bad_alloc();
    if (void* p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main() {
    constexpr size_t kChunks = 40, kBytes = 4096;
    static char from[kChunks * kBytes], to[kChunks * kBytes];
    for (size_t i = 0; i < sizeof(from); ++i) from[i] = (char)(i * 31 + i / kBytes);
    int threw = 0;
    for (long fail = -1; fail < 30; ++fail) {
        std::memset(to, 0, sizeof(to));
        left = fail;
        try {
            od::CopyCrew crew(kChunks);
            crew.begin();
            for (size_t c = 0; c < kChunks; ++c) crew.give(c, to + c * kBytes, from + c * kBytes, kBytes);
            for (size_t c = 0; c < kChunks; ++c) crew.wait(c);
            left = -1;
            if (std::memcmp(from, to, sizeof(to)) != 0) return 2;
        } catch (const std::bad_alloc&) {
            ++threw;
        }
        left = -1;
    }
    std::printf("threw %d\n", threw);
    return threw > 0 && threw < 30 ? 0 : 3;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_allocation_may_fail(tmp_path):
    src, exe = tmp_path / "crew.cpp", tmp_path / "crew"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, (p.returncode, p.stdout, p.stderr)
