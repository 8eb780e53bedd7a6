"""The divisions of the kernels' index arithmetic (csrc/fastdiv.hpp), compiled for the host: where exact() says so every quotient is
right, and where it refuses some quotient is wrong.  Divisors that networks bring (pixels of a flattened image, rows of tall
images, channels) and random ones."""
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "fastdiv.hpp"
// stdin: divisor, largest dividend.  Looks at n = k d - 1 (a wrong multiplier is off in front of a multiple first), k d and the
// largest dividend, for up to 200 000 multiples from the last one downwards.  Prints what exact() says and whether a quotient is off.
int main() {
  long long d, most;
  while (scanf("%lld %lld", &d, &most) == 2) {
    sasgd::FastDiv f;
    f.set((int)d);
    bool off = f((int)most) != most / d;
    long long k = (most + 1) / d;
    for (int i = 0; i < 200000 && k >= 1; i++, k--) {
      off = off || f((int)(k * d - 1)) != k - 1;
      off = off || (k * d <= most && f((int)(k * d)) != k);
    }
    printf("%d %d\n", (int)sasgd::FastDiv::exact((int)d, most), (int)off);
  }
  return 0;
}
"""


def divisor_pairs():
    pairs = []
    for channels, side in ((8, 160), (8, 224), (64, 112), (32, 128), (24, 150), (3, 1000), (16, 200), (64, 7), (1, 1), (5, 3)):
        pairs += [(side * side, channels * side * side - 1), (channels, channels * side * side - 1), (side, side * side - 1)]
    for h, w in ((7000, 800), (1100, 2000), (40_000, 600)):       # tall images: h w w beyond 2^32
        pairs += [(w, h * w - 1), (w + 4, 16_383)]
    return pairs


def test_exact_says_where_quotients_are_right(tmp_path):
    src, exe = tmp_path / "divide.cpp", tmp_path / "divide"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(src), "-o", str(exe)])
    rng = np.random.default_rng(0)
    pairs = divisor_pairs()
    pairs += [(int(2 ** rng.uniform(0, 31)), int(2 ** rng.uniform(0, 31)) - 1) for _ in range(2000)]
    pairs += [(d, min(2 ** 31 - 1, 2 ** 32 // d - 1)) for d in range(1, 2000)]          # the range that always holds
    out = subprocess.check_output([str(exe)], input="\n".join("%d %d" % p for p in pairs), text=True).split("\n")
    said = [tuple(map(int, line.split())) for line in out if line]
    assert len(said) == len(pairs)
    for (d, most), (exact, off) in zip(pairs, said):
        assert exact != off, (d, most, exact, off)
        if d * (most + 1) <= 2 ** 32:
            assert exact, (d, most)
    refused = {p: s[0] for p, s in zip(pairs, said)}
    assert not refused[(160 * 160, 8 * 160 * 160 - 1)] and not refused[(112 * 112, 64 * 112 * 112 - 1)]
