"""The byte-overlap test of the update calls (host code) against a comparison of every pair of blocks, over random views
of one allocation (equal strides, the solved form), other strides, zero strides and single blocks."""
import os
import subprocess

import pytest

from paper_2510_12872_amd import build

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "kvcomm_device.h"
using namespace kvc;
static int64_t rnd(int64_t n) { return (int64_t)(((uint64_t)rand() << 31 | (uint64_t)rand()) % (uint64_t)n); }
static bool brute(const Extent &a, const Extent &b)
{
    for (int l = 0; l < a.L; ++l) for (int h = 0; h < a.H; ++h)
        for (int m = 0; m < b.L; ++m) for (int g = 0; g < b.H; ++g) {
            const int64_t x = (int64_t)a.base + l * a.sl + h * a.sh, y = (int64_t)b.base + m * b.sl + g * b.sh;
            if (x < y + b.run && y < x + a.run) return true;
        }
    return false;
}
int main()
{
    srand(1);
    long yes = 0, no = 0;
    for (int it = 0; it < 200000; ++it) {
        Extent a, b;
        a.L = 1 + rnd(5); a.H = 1 + rnd(5);
        const bool same = rnd(4) != 0;
        const int64_t tok = 1 + rnd(6), cap = 1 + rnd(12);
        a.run = tok * (1 + rnd(cap));
        a.sh = rnd(8) ? tok * cap * (rnd(3) ? 1 : a.L) : rnd(40);
        a.sl = rnd(8) ? (rnd(2) ? a.sh * a.H : tok * cap) : rnd(60);
        a.base = 4096 + rnd(64);
        b = a;
        if (!same) { b.L = 1 + rnd(5); b.H = 1 + rnd(5); b.sh = rnd(40); b.sl = rnd(60); }
        b.run = tok * (1 + rnd(cap));
        b.base = a.base - 200 + rnd(400);
        const bool want = brute(a, b), got = extents_overlap(a, b);
        if (want != got) {
            printf("a base %lld sl %lld sh %lld run %lld L %d H %d  b base %lld sl %lld sh %lld run %lld L %d H %d: want %d got %d\n",
                   (long long)a.base, (long long)a.sl, (long long)a.sh, (long long)a.run, a.L, a.H, (long long)b.base,
                   (long long)b.sl, (long long)b.sh, (long long)b.run, b.L, b.H, want, got);
            return 1;
        }
        (want ? yes : no)++;
    }
    printf("%ld overlap, %ld do not\n", yes, no);
    return yes < 20000 || no < 20000;
}
"""


def test_extents_overlap_against_every_pair_of_blocks(tmp_path):
    src, exe = tmp_path / "extents.hip", tmp_path / "extents"
    src.write_text(MAIN)
    cmd = [build.hipcc_path(), "--cuda-host-only", "-O2", "-std=c++17", "-I", os.path.join(build.ROOT, "include"), "-I",
           build.CSRC, "-o", str(exe), str(src)]
    made = subprocess.run(cmd, capture_output=True, text=True)
    if made.returncode:
        pytest.fail(made.stderr[-2000:])
    ran = subprocess.run([str(exe)], capture_output=True, text=True)
    assert ran.returncode == 0, ran.stdout
