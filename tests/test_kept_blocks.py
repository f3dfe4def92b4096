"""The device memory that a ctx keeps between hierarchy builds, over an
allocator of 100 bytes: an allocation that would fail gets back the blocks that
no build under way uses, in a build's first phase the second's, and outside of
a build both; blocks in use stay."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2406_12080_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include "kept_blocks.h"
using hgs::KeptBlocks;
static std::map<void *, size_t> held;
static size_t used = 0;
static int take(void **p, size_t n)
{
    if (used + n > 100) return 2;
    *p = std::malloc(n);
    held[*p] = n;
    used += n;
    return 0;
}
static void give(void *p)
{
    if (!held.count(p)) std::abort();
    used -= held[p];
    held.erase(p);
    std::free(p);
}
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s, %zu used\n", __LINE__, #x, used); return 1; } } while (0)
int main()
{
    {
        KeptBlocks k(take, give);
        size_t n;
        void *p, *q;
        // a build whose blocks stay
        CHECK(k.reserve(0, 30, n) && n == 30);
        CHECK(k.reserve(1, 40, n) && n == 40);
        CHECK(k.alloc(&p, 31) == 2 && !p && used == 70);  // nothing idle to give back
        k.release(50);
        CHECK(used == 70);
        // the next: the same block again, and what its first phase lacks from the second's
        char *b = k.reserve(0, 20, n);
        CHECK(b && n == 30 && used == 70);
        CHECK(k.alloc(&p, 50) == 0 && used == 80);
        CHECK(!k.reserve(1, 40, n) && n == 0 && used == 80);  // no room: one by one
        CHECK(k.alloc(&q, 20) == 0 && used == 100);
        give(p);
        give(q);
        k.release(50);
        CHECK(used == 30);
        // a larger first block takes the room of the second
        CHECK(k.reserve(1, 60, n) && used == 90);
        k.release(60);
        CHECK(used == 90);
        CHECK(k.reserve(0, 50, n) && n == 50 && used == 50);
        k.release(60);
        // beyond the limit it goes
        CHECK(k.reserve(1, 50, n) && used == 100);
        k.release(49);
        CHECK(used == 0);
        // any other allocation gets both back
        CHECK(k.reserve(0, 30, n) && k.reserve(1, 30, n));
        k.release(50);
        CHECK(k.alloc(&p, 100) == 0 && used == 100);
        give(p);
        CHECK(k.alloc(&p, 101) == 2 && used == 0);
        CHECK(k.reserve(0, 30, n));
        k.release(50);
    }
    CHECK(used == 0);  // the ctx's end
    return 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no host compiler")
def test_blocks_are_given_back(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
