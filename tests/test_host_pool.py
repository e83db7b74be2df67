"""The bounded pool of staging buffers, on the host: no more than its number are made, a
caller that finds all of them out gets none and does not wait, a failed allocation takes no
place, and all are given back at the end.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include "host_copy.h"
int main() {
    eifp::BufferPool<3> pool;
    std::atomic<int> made{0}, freed{0};
    auto alloc = [&]() -> void* { ++made; return std::malloc(64); };
    auto none = []() -> void* { return nullptr; };
    if (pool.take(none)) return 1;
    void* a = pool.take(alloc);
    void* b = pool.take(alloc);
    if (pool.take(none)) return 2;  // the last place stays free
    void* c = pool.take(alloc);
    if (!a || !b || !c || pool.take(alloc) || made != 3) return 3;
    std::atomic<int> got{0};
    std::thread other([&] { got = pool.take(alloc) ? 1 : -1; });  // all out: returns, with none
    other.join();
    if (got != -1) return 4;
    pool.give(b);
    if (pool.take(alloc) != b || made != 3) return 5;
    pool.give(a), pool.give(b), pool.give(c);
    // many users: a buffer is one user's at a time
    std::atomic<int> wrong{0}, without{0};
    std::vector<std::thread> ts;
    for (int t = 0; t < 8; ++t)
        ts.emplace_back([&, t] {
            for (int i = 0; i < 20000; ++i) {
                volatile int* p = (volatile int*)pool.take(alloc);
                if (!p) { ++without; continue; }
                p[0] = t;
                for (int k = 0; k < 16; ++k) p[1] = k;
                if (p[0] != t) ++wrong;
                pool.give((void*)p);
            }
        });
    for (auto& t : ts) t.join();
    if (wrong || made != 3) return 6;
    pool.release([&](void* p) { ++freed; std::free(p); });
    if (freed != 3) return 7;
    printf("%d calls without a buffer\n", without.load());
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_buffer_pool_is_bounded_and_never_waits(tmp_path):
    src, exe = tmp_path / "h.cpp", tmp_path / "h"
    src.write_text(HARNESS)
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I",
                        os.path.join(ROOT, "paper_2210_06232_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(out.stdout)
    assert out.returncode == 0, out.returncode
