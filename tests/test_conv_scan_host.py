"""The patch rows that a convolution's tiles need, without a GPU: the scan over one period of tiles against a count
over every tile, position by position."""

import math
import os
import random
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include "conv_scan.h"
int main() {
  long m, hwo, wo, sh, kh, tp;
  while (std::scanf("%ld %ld %ld %ld %ld %ld", &m, &hwo, &wo, &sh, &kh, &tp) == 6) {
    int64_t looked;
    const int rows = gs::scan_patch_rows(m, hwo, wo, sh, kh, tp, 16, &looked);
    std::printf("%d %ld\n", rows, long(looked));
  }
}
"""


def every_tile(m, ho, wo, sh, kh, tp):
    """Rows between the first and the last output row, times the stride, plus a window, per image of a tile."""
    pos = np.arange(m)
    image, row = pos // (ho * wo), pos % (ho * wo) // wo
    most = 0
    for first in range(0, m, tp):
        i, r = image[first:first + tp], row[first:first + tp]
        if i[-1] - i[0] + 1 > 16:
            return -1
        need = sum((r[i == k].max() - r[i == k].min()) * sh + kh for k in range(i[0], i[-1] + 1))
        most = max(most, int(need))
    return most


def test_scan_of_one_period(tmp_path):
    src, exe = tmp_path / "scan.cpp", tmp_path / "scan"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2105_09377_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    rng = random.Random(2105)
    # planes smaller and larger than a tile, of one row and of one column, tiles that divide a plane, whole and cut last tiles
    cases = [(1, 1, 1, 1, 1, 32), (64, 1, 1, 2, 3, 32), (33, 1, 1, 1, 3, 32), (7, 7, 7, 1, 3, 56), (64, 56, 56, 1, 3, 128), (3, 8, 4, 1, 3, 96)]
    cases += [(rng.randint(1, 60), rng.randint(1, 30), rng.randint(1, 30), rng.randint(1, 3), rng.randint(1, 5),
               8 * rng.randint(1, 32)) for _ in range(300)]
    text = "".join(f"{n * ho * wo} {ho * wo} {wo} {sh} {kh} {tp}\n" for n, ho, wo, sh, kh, tp in cases)
    out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True).stdout.split()
    for (n, ho, wo, sh, kh, tp), rows, looked in zip(cases, out[::2], out[1::2]):
        assert int(rows) == every_tile(n * ho * wo, ho, wo, sh, kh, tp), (n, ho, wo, sh, kh, tp)
        assert int(looked) <= ho * wo // math.gcd(ho * wo, tp) + 1
