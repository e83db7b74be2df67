"""First touches of large output arrays, on the host: a fresh array has all its pages after
them, and an array that has its pages already is not written to (its pages are made
read-only here, so a write would end the harness).
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <cstdio>
#include <cstring>
#include <sys/mman.h>
#include "host_copy.h"
int main() {
    const long long bytes = (40LL << 20) + 4096 * 3;  // above the size from which pages are touched
    char* p = (char*)mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (p == (char*)MAP_FAILED) return 2;
    madvise(p, bytes, MADV_NOHUGEPAGE);
    auto missing = [&] {
        std::vector<unsigned char> in(bytes / 4096);
        mincore(p, bytes, in.data());
        long long m = 0;
        for (unsigned char x : in) m += !(x & 1);
        return m;
    };
    const long long before = missing();
    eifp::touch_pages(p, bytes);
    const long long after = missing();
    std::memset(p, 7, bytes);
    mprotect(p, bytes, PROT_READ);
    eifp::touch_pages(p, bytes);         // nothing to fault in: no write
    eifp::touch_pages(p + 5, bytes - 9);  // nor for an array that starts inside a page
    printf("%lld %lld\n", before, after);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_touch_pages_faults_fresh_arrays_in_and_leaves_others_alone(tmp_path):
    src, exe = tmp_path / "h.cpp", tmp_path / "h"
    src.write_text(HARNESS)
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I",
                        os.path.join(ROOT, "paper_2210_06232_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.returncode
    before, after = map(int, out.stdout.split())
    assert before > 10000 and after == 0
