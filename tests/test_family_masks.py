"""The index logic of the plane writers (csrc/mt_masks.h) on the host, under
the undefined-behaviour sanitizer: the walk over a mask's powers ends at its
highest one, also for a family of 32 powers (the most the ABI accepts), writes
every wanted power once, in ascending order, and visits none outside the
family."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1511_05690_amd", "csrc")

PROGRAM = r"""
#include "mt_masks.h"
#include <cstdio>
static int check(uint32_t mask, int n_p) {
    mask &= mt::family_bits(n_p);
    uint32_t written = 0;
    int visited = 0, bad = 0;
    mt::each_power(mask, [&](int q, bool wanted) {
        if (++visited > 40) __builtin_trap();
        bad |= q != visited - 1 || q >= n_p;
        if (wanted) {
            bad |= (written >> q) != 0u;
            written |= 1u << q;
        }
    });
    bad |= written != mask || (mask != 0u && ((mask >> (visited - 1)) & 1u) == 0u) || (mask == 0u && visited != 0);
    if (bad) printf("mask %08x of %d powers: wrote %08x, visited %d\n", mask, n_p, written, visited);
    return bad;
}
int main() {
    int bad = 0;
    uint32_t r = 12345u;
    for (int n_p = 1; n_p <= 32; ++n_p) {
        bad |= check(~0u, n_p) | check(0u, n_p) | check(~3u, n_p) | check(3u, n_p) | check(7u << (n_p > 3 ? n_p - 3 : 0), n_p);
        for (int q = 0; q < n_p; ++q) bad |= check(1u << q, n_p) | check(~(1u << q), n_p);
        for (int t = 0; t < 200; ++t) bad |= check(r = r * 1664525u + 1013904223u, n_p);
    }
    return bad;
}
"""


def test_walk_over_the_powers(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
