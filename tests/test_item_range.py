"""Host-side checks of the particles of a leaf's work items.

A tree layout cuts a leaf's particles into ceil(n / 16) items
(csrc/item_range.h). A small C++ program, built here with g++ against that header,
checks that the items of a leaf follow one another from its first particle to its
last with 1 to 16 particles each, for every leaf size up to 4,096 and for sizes at
which 32-bit products overflow, up to the largest particle count the library
accepts; and that the form without a division agrees where the walks use it."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1508_00115_amd", "csrc")

PROGRAM = r"""
#include "item_range.h"
#include <cstdio>
#include <initializer_list>

static int check(int ni)
{
    const int nt = (int)(((long long)ni + 15) / 16);
    if (item_first(ni, nt, 0) != 0 || item_first(ni, nt, nt) != ni) return std::printf("ends of %d\n", ni), 1;
    // every item of small leaves; of large ones the first, the last and one in a thousand
    for (int t = 0; t < nt; t += nt > 4096 && t > 64 && t + 1064 < nt ? 1000 : 1) {
        const int n = item_first(ni, nt, t + 1) - item_first(ni, nt, t);
        if (n < 1 || n > 16) return std::printf("item %d of %d holds %d\n", t, ni, n), 1;
        if (nt <= 4 && item_first_small(ni, nt, t) != item_first(ni, nt, t)) return std::printf("small %d\n", ni), 1;
    }
    return nt <= 4 && item_first_small(ni, nt, nt) != ni;
}

int main()
{
    int bad = 0;
    for (int ni = 1; ni <= 4096; ++ni) bad += check(ni);
    for (int ni : {185362, 185363, 185379, 262144, 1000003, 16777216, 100000007, 2147483646}) bad += check(ni);
    return bad != 0;
}
"""


def test_items_cover_a_leaf(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src = tmp_path / "items.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "items"
    subprocess.run([gxx, "-std=c++17", "-O1", "-ftrapv", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
