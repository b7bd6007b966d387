"""Order in which a launch's blocks take its tiles (xcd_order): every tile once,
and for any number of blocks those of one XCD (b % 8) take one contiguous range
in launch order, so that tiles sharing a halo meet in one L2."""
import os
import subprocess

from paper_2106_07694_amd import build

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "lbw_internal.h"
int main() {
    for (int nb = 1; nb < 3000; nb += nb < 200 ? 1 : 37) {
        std::vector<int> seen(nb, 0);
        int next = 0;
        for (int xcd = 0; xcd < 8; ++xcd)
            for (int b = xcd; b < nb; b += 8) {
                const int t = lbw::xcd_order(b, nb);
                if (t != next++ || t < 0 || t >= nb || seen[t]++) { printf("%d blocks: block %d takes %d\n", nb, b, t); return 1; }
            }
        if (next != nb) return 1;
    }
    // a work list walked by as many blocks as it has items: one item each
    for (int n = 8; n < 2000; ++n)
        for (int xcd = 0; xcd < 8; ++xcd) {
            const int blocks = n / 8 + (xcd < n % 8);
            if (lbw::xcd_first(xcd + 1, n) - lbw::xcd_first(xcd, n) != blocks || lbw::xcd_first(0, n) != 0 ||
                lbw::xcd_first(8, n) != n) { printf("%d items, XCD %d\n", n, xcd); return 1; }
        }
    const int big = 0x7fffffff;      // the largest launch: no overflow
    return lbw::xcd_order(big - 1, big) == big - 1 - (big >> 3) ? 0 : 1;
}
"""


def test_each_xcd_takes_a_contiguous_range(tmp_path):
    src, exe = tmp_path / "order.hip", tmp_path / "order"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, "-std=c++17", "-O1", "--cuda-host-only", "-I", build.CSRC, "-x", "hip", str(src),
                    "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
