"""PinnedPool (csrc/df_pinned.hpp), the page-locked buffers of df_iterate's readbacks, with a
counting allocator: repeated calls of one size allocate once, also above 256 KiB (64
instances read back 524 KB); what is kept is bounded; threads never share a buffer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <thread>
#include <vector>
#include "df_pinned.hpp"
static std::atomic<int> n_alloc{0}, n_free{0};
static bool fail = false;
static void *get(size_t b) { if (fail) return nullptr; ++n_alloc; return malloc(b); }
static void put(void *p) { ++n_free; free(p); }
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    size_t c;
    for (size_t bytes : {100ul, 262144ul, 262145ul, 524288ul + 4096, 4ul << 20}) {
        df::PinnedPool p(get, put);
        n_alloc = n_free = 0;
        for (int i = 0; i < 5; ++i) {
            void *b = p.take(bytes, &c);
            CHECK(b && c >= bytes);
            memset(b, 1, bytes);
            p.give(b, c);
        }
        CHECK(n_alloc == 1 && n_free == 0);
    }
    {   // larger ones are not kept
        df::PinnedPool p(get, put);
        n_alloc = n_free = 0;
        for (int i = 0; i < 3; ++i) { void *b = p.take((4ul << 20) + 1, &c); p.give(b, c); }
        CHECK(n_alloc == 3 && n_free == 3);
    }
    {   // a large buffer serves small calls; large ones push small ones out; 8 MiB, 8 buffers
        df::PinnedPool p(get, put);
        n_alloc = n_free = 0;
        void *b[12]; size_t cap[12];
        for (int i = 0; i < 12; ++i) b[i] = p.take(1000, &cap[i]);
        for (int i = 0; i < 12; ++i) p.give(b[i], cap[i]);
        CHECK(n_alloc == 12 && n_free == 4);
        for (int i = 0; i < 3; ++i) b[i] = p.take(4ul << 20, &cap[i]);
        for (int i = 0; i < 3; ++i) p.give(b[i], cap[i]);
        CHECK(n_alloc - n_free <= 8);
        n_alloc = 0;
        void *x = p.take(4ul << 20, &c); size_t d; void *y = p.take(1000, &d);
        CHECK(n_alloc == 0 && x != y);
    }
    {
        df::PinnedPool p(get, put);
        fail = true;
        CHECK(p.take(10, &c) == nullptr);
        fail = false;
    }
    df::PinnedPool p(get, put);
    std::atomic<int> bad{0};
    std::vector<std::thread> t;
    for (int k = 0; k < 8; ++k)
        t.emplace_back([&, k] {
            for (int i = 0; i < 2000; ++i) {
                size_t cap;
                const size_t n = 1000 + 300000 * ((i + k) % 3);
                char *b = (char *)p.take(n, &cap);
                b[0] = (char)k; b[n - 1] = (char)k;
                std::this_thread::yield();
                if (b[0] != k || b[n - 1] != k) ++bad;
                p.give(b, cap);
            }
        });
    for (auto &x : t) x.join();
    CHECK(bad == 0);
    return 0;
}
"""


def test_pool(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    inc = os.path.join(ROOT, "paper_1507_00895_amd", "csrc")
    subprocess.run([cxx, "-O1", "-std=c++17", "-pthread", "-I", inc, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout)
