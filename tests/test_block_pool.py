"""The pool of idle device blocks (csrc/block_pool.h) on the CPU, with a counting
allocator in the driver's place: its bounds, the eviction of blocks that are
passed over, the memory given back when an allocation fails, and threads that
take and return blocks at once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "block_pool.h"
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <thread>
#include <vector>
using namespace rorbk;

// allocator of at most g_limit bytes in use; small blocks are real memory
static std::atomic<size_t> g_used{0}, g_calls{0};
static size_t g_limit = (size_t)-1;
struct Head { size_t bytes; };
static int get_mem(void **p, size_t bytes) {
    ++g_calls;
    if (g_used.fetch_add(bytes) + bytes > g_limit) { g_used -= bytes; return 2; }
    Head *h = (Head *)malloc(sizeof(Head) + (bytes < 4096 ? bytes : 4096));
    h->bytes = bytes;
    *p = h + 1;
    return 0;
}
static void free_mem(void *p) {
    Head *h = (Head *)p - 1;
    g_used -= h->bytes;
    free(h);
}
#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
static const size_t MB = 1 << 20;

int main() {
    {   // kept blocks come back to requests of at least half their size, same device
        BlockPool pool(get_mem, free_mem);
        Block b, c;
        CHECK(pool.get(&b, 100 * MB, 0) == 0 && b.bytes == 100 * MB);
        char *p = b.p;
        pool.put(&b);
        CHECK(!b.p && g_used == 100 * MB);
        CHECK(pool.get(&c, 100 * MB, 1) == 0 && c.p != p);      // another device
        CHECK(pool.get(&b, 49 * MB, 0) == 0 && b.p != p);       // too large for it
        Block d;
        CHECK(pool.get(&d, 60 * MB, 0) == 0 && d.p == p && d.bytes == 100 * MB);
        free_mem(b.p); free_mem(c.p); free_mem(d.p);
        CHECK(g_used == 0);
    }
    {   // bounds: MAX_BLOCKS blocks, MAX_BYTES bytes
        BlockPool pool(get_mem, free_mem);
        Block b[12];
        for (int i = 0; i < 12; ++i) CHECK(pool.get(&b[i], MB, 0) == 0);
        for (int i = 0; i < 12; ++i) pool.put(&b[i]);
        CHECK(g_used == BlockPool::MAX_BLOCKS * MB);
        CHECK(pool.trim() == BlockPool::MAX_BLOCKS && g_used == 0 && pool.trim() == 0);
        for (int i = 0; i < 3; ++i) CHECK(pool.get(&b[i], 900 * MB, 0) == 0);
        for (int i = 0; i < 3; ++i) pool.put(&b[i]);
        CHECK(g_used == 1800 * MB);
        CHECK(pool.get(&b[0], BlockPool::MAX_BYTES + 1, 0) == 0);
        pool.put(&b[0]);                                        // never kept
        CHECK(g_used == 1800 * MB);
        pool.trim();
        CHECK(g_used == 0);
    }
    {   // a block passed over MAX_MISSES times goes back; one that is used does not
        BlockPool pool(get_mem, free_mem);
        Block big, b;
        CHECK(pool.get(&big, 500 * MB, 0) == 0);
        pool.put(&big);
        for (int i = 0; i < BlockPool::MAX_MISSES; ++i) {
            CHECK(g_used >= 500 * MB);
            CHECK(pool.get(&b, MB, 0) == 0);
            pool.put(&b);
        }
        CHECK(g_used == MB);
        const size_t calls = g_calls;
        for (int i = 0; i < 100; ++i) { CHECK(pool.get(&b, MB, 0) == 0); pool.put(&b); }
        CHECK(g_calls == calls);
        pool.trim();
    }
    {   // memory used up: idle blocks are given back to alloc and to get alike
        BlockPool pool(get_mem, free_mem);
        g_limit = 1000 * MB;
        Block b;
        void *p = nullptr;
        CHECK(pool.get(&b, 800 * MB, 0) == 0);
        CHECK(pool.alloc(&p, 300 * MB) == 2);                   // in use, not idle
        pool.put(&b);
        CHECK(pool.alloc(&p, 300 * MB) == 0 && g_used == 300 * MB);
        CHECK(pool.get(&b, 600 * MB, 0) == 0);
        pool.put(&b);
        Block c;
        CHECK(pool.get(&c, 250 * MB, 0) == 0 && c.p && g_used == 550 * MB);   // 600 > 2 x 250
        pool.put(&c);
        CHECK(pool.get(&c, 2000 * MB, 0) == 2 && !c.p && g_used == 300 * MB);
        free_mem(p);
        g_limit = (size_t)-1;
    }
    {   // threads: a block in use belongs to one of them
        BlockPool pool(get_mem, free_mem);
        std::atomic<int> bad{0};
        std::vector<std::thread> ts;
        for (int t = 0; t < 8; ++t)
            ts.emplace_back([&pool, &bad, t] {
                for (int i = 0; i < 4000; ++i) {
                    Block b;
                    if (pool.get(&b, 256 + 64 * ((t + i) % 5), 0) != 0) { ++bad; return; }
                    memset(b.p, t, 256);
                    if (i % 64 == 0) std::this_thread::yield();
                    for (int k = 0; k < 256; ++k) bad += b.p[k] != (char)t;
                    if (i % 97 == 0) pool.trim();
                    pool.put(&b);
                }
            });
        for (auto &t : ts) t.join();
        CHECK(bad == 0);
        pool.trim();
        CHECK(g_used == 0);
    }
    printf("ok\n");
    return 0;
}
"""


def test_block_pool(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "pool.cpp", tmp_path / "pool"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread",
                    "-I" + os.path.join(ROOT, "paper_2510_02156_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
