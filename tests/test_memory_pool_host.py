"""The pool of kept device memory (csrc/memory_pool.h), compiled by the host compiler: what
it takes beyond a request, its bound, the oldest block leaving first, one device's blocks
not serving another, and a host that runs out of memory at every point in turn."""
import os
import subprocess

import pytest

from paper_2507_11094_amd import build

CODE = r"""
#include <cassert>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <set>
#include <vector>

static long left = -1;  // allocations that still succeed; < 0: all
void *operator new(size_t n) {
    if (left == 0) throw std::bad_alloc();
    if (left > 0) --left;
    if (void *p = malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

#include "memory_pool.h"

static bool live[4096];  // device blocks
static int made = 1;
static void *dev_alloc() { live[made] = true; return (void *)(size_t)(made++ << 8); }
static void dev_free(void *p) {
    const size_t i = (size_t)p >> 8;
    assert(i && live[i]);
    live[i] = false;
}
static int live_count() {
    int c = 0;
    for (bool b : live) c += b;
    return c;
}
typedef dg::MemoryPool Pool;
static void *get(Pool &q, size_t bytes, int dev = 0) {
    void *p = q.take(bytes, dev);
    if (p) return p;
    p = dev_alloc();
    q.note(p, bytes, dev);
    return p;
}
static void put(Pool &q, void *p, bool keep) {
    if (!q.give(p, keep)) dev_free(p);
}

int main(int, char **a) {
    if (a[1][0] == 'r') {
        for (size_t n = 1; n < ((size_t)1 << 40); n += 1 + n / 7) {
            const size_t r = Pool::round(n);
            assert(r >= n && r - n < (64 << 10) && r - n <= 256 + n / 8);
        }
    } else if (a[1][0] == 'b') {
        Pool q(1000, dev_free);
        void *x = get(q, 400), *y = get(q, 500), *z = get(q, 450), *big = get(q, 1001);
        put(q, x, true), put(q, y, true), put(q, big, true);
        assert(live_count() == 3);   // more than the bound is not kept
        put(q, z, true);             // 1,350 bytes: the oldest leaves
        assert(live_count() == 2 && !live[(size_t)x >> 8]);
        assert(q.take(500, 1) == nullptr && q.take(300, 0) == nullptr);
        assert(q.take(420, 0) == z && q.take(420, 0) == y && q.take(1, 0) == nullptr);
        put(q, y, false), put(q, z, true);
        q.trim();
        assert(live_count() == 0);
    } else {
        for (long k = 0; k < 60; ++k) {  // the k-th allocation of the host and all later ones fail
            Pool q(1000, dev_free);
            left = k;
            void *p[8];
            for (int i = 0; i < 8; ++i) p[i] = get(q, 100 + i);
            for (int i = 0; i < 8; ++i) put(q, p[i], i != 3);
            for (int i = 0; i < 8; ++i) p[i] = get(q, 100 + i, i == 5);
            for (int i = 0; i < 8; ++i) put(q, p[i], true);
            q.trim();
            left = -1;
            assert(live_count() == 0);
        }
    }
    puts("ok");
}
"""


@pytest.fixture(scope="module")
def prog(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool")
    (d / "p.cpp").write_text(CODE)
    subprocess.check_call(["g++", "-std=c++17", "-pthread", "-I", build.CSRC, str(d / "p.cpp"), "-o", str(d / "p")])
    return str(d / "p")


@pytest.mark.parametrize("part", ["round", "bound", "host memory"])
def test_pool(prog, part):
    assert subprocess.check_output([prog, part]) == b"ok\n"
