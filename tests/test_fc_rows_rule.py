"""The rule by which a fully connected layer's tiles and splits are chosen (csrc/tile_rules.hpp), compiled for the host."""
import os
import subprocess

import pytest

pytest.importorskip("torch")
import test_gpu_fc_rows as rows            # noqa: E402  (the networks; nothing runs on a GPU here)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "tile_rules.hpp"
int main() {
  int K, N, rows, groups;
  size_t scratch;
  while (scanf("%d %d %d %d %zu", &K, &N, &rows, &groups, &scratch) == 5) {
    const sasgd::FcRowsChoice c = sasgd::fc_rows_choice(K, N, rows, groups, scratch);
    printf("%d %d\n", c.tm, c.splits);
  }
}
"""
SCRATCH = 128 << 20


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)

    def run(queries):
        out = subprocess.run([str(d / "rule")], input="\n".join(" ".join(map(str, q)) for q in queries), capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def test_choices_are_valid(ask):
    queries = [(K, N, r, g, s) for K in (8, 64, 72, 1000, 4096, 9216) for N in (8, 104, 1000, 9216) for r in (1, 64, 65, 129, 256, 288, 2048, 262144)
               for g in (1, 7, 64) for s in (0, 1 << 20, SCRATCH, 1 << 33)]
    for (K, N, r, g, s), (tm, sp) in zip(queries, ask(queries)):
        steps = -(-K // 64)
        assert 1 <= tm <= 4 and (tm == 1 or 64 * (tm - 1) < r)
        assert 1 <= sp <= 16
        if sp > 1:
            assert -(-steps // -(-steps // sp)) == sp          # no workgroup without a stage
            assert sp * r * N * 4 <= s and r * N * 4 < 2 ** 31   # the partial sums have room, and 32-bit offsets


def test_the_gpu_cases_reach_every_height(ask):
    seen = set()
    for name, (net, mu, lam, want) in rows.CASES.items():
        K, N = (1152, 3080) if net is rows.WIDE else (72, 200)
        for (tm, sp), form in zip(ask([(K, N, mu * lam, 1, SCRATCH), (N, K, mu * lam, 1, SCRATCH)]), want):
            assert (tm, sp > 1) == form, (name, tm, sp)
            seen.add((tm, sp > 1))
    assert {(1, True), (1, False), (2, False), (3, False), (3, True), (4, False)} <= seen


# Measured on one card, us with the second pass: K, N, rows, versions; {(height, splits): us} of the fastest forms, and of the kernels before
MEASURED = [
    (9216, 4096, 16, 1, {(1, 1): 44.0, (1, 2): 29.6, (1, 3): 22.8, (1, 4): 20.2, (1, 5): 18.6, (1, 6): 19.0, (1, 8): 18.4, (1, 10): 20.0, (1, 12): 19.7, (1, 16): 19.2}, 20.2),
    (4096, 9216, 16, 1, {(1, 1): 24.9, (1, 2): 19.7, (1, 3): 18.4, (1, 4): 22.4, (1, 5): 20.5, (1, 6): 20.5, (1, 8): 22.2, (1, 10): 21.6, (1, 12): 23.3, (1, 16): 23.6}, 21.0),
    (9216, 4096, 64, 1, {(1, 1): 46.4, (1, 2): 30.7, (1, 3): 23.7, (1, 4): 21.0, (1, 5): 19.9, (1, 6): 19.2, (1, 8): 19.5, (1, 10): 22.0, (1, 12): 20.6, (1, 16): 20.8}, 35.6),
    (4096, 4096, 128, 1, {(1, 2): 25.7, (1, 3): 21.5, (1, 4): 19.7, (1, 5): 23.8, (1, 6): 23.9, (1, 8): 22.2, (2, 3): 25.0, (2, 4): 21.2, (2, 5): 20.2, (2, 6): 22.2, (2, 8): 22.0, (2, 10): 25.6, (2, 12): 24.5, (2, 16): 26.9}, 39.2),
    (9216, 4096, 256, 1, {(1, 2): 34.3, (1, 3): 36.4, (1, 4): 33.4, (1, 5): 37.8, (1, 6): 35.7, (1, 8): 38.8, (2, 3): 34.2, (2, 4): 31.0, (2, 6): 37.8, (2, 8): 37.6, (3, 4): 36.6, (4, 5): 37.6, (4, 6): 36.0, (4, 8): 35.4}, 62.2),
    (4096, 4096, 256, 1, {(1, 2): 23.6, (1, 4): 27.2, (2, 2): 30.6, (2, 3): 26.2, (2, 4): 23.0, (2, 8): 31.0, (3, 2): 29.9, (3, 3): 25.8, (3, 4): 24.2, (4, 3): 30.1, (4, 4): 27.5, (4, 5): 26.6, (4, 6): 25.4, (4, 8): 27.3}, 50.2),
    (4096, 9216, 256, 1, {(1, 3): 55.2, (2, 1): 48.0, (2, 2): 55.5, (2, 3): 48.0, (2, 4): 54.8, (2, 5): 52.6, (3, 1): 50.1, (3, 3): 49.8, (3, 5): 55.2, (4, 2): 41.5, (4, 3): 36.8, (4, 4): 51.8, (4, 5): 50.0, (4, 6): 50.6}, 78.3),
    (9216, 4096, 288, 1, {(1, 1): 50.6, (1, 3): 41.0, (1, 4): 45.6, (1, 5): 45.0, (1, 6): 46.9, (1, 8): 50.6, (2, 2): 44.0, (2, 4): 47.6, (2, 5): 45.8, (3, 3): 43.0, (3, 4): 38.6, (3, 5): 51.0, (3, 8): 47.2, (4, 4): 45.3}, 107.0),
    (4096, 9216, 288, 1, {(1, 1): 40.9, (1, 2): 43.0, (1, 3): 50.1, (1, 4): 47.4, (1, 5): 52.9, (2, 1): 40.2, (2, 2): 46.6, (2, 3): 52.0, (2, 4): 54.4, (3, 1): 50.6, (3, 2): 55.6, (3, 3): 48.0, (3, 4): 54.7, (3, 5): 53.9}, 71.2),
    (4096, 4096, 576, 1, {(1, 1): 40.3, (1, 2): 42.4, (1, 3): 41.8, (1, 4): 43.0, (1, 5): 45.0, (2, 1): 41.4, (2, 2): 45.3, (2, 3): 40.8, (2, 4): 45.7, (3, 2): 35.9, (3, 3): 46.3, (3, 4): 41.7, (3, 5): 42.8, (4, 2): 41.6}, 64.7),
    (9216, 4096, 16, 7, {(1, 1): 103.8, (1, 2): 104.8, (1, 3): 106.7, (1, 4): 108.9, (1, 5): 107.4, (1, 6): 113.6, (1, 8): 107.7, (1, 10): 112.1, (1, 12): 110.7, (1, 16): 117.1}, 115.1),
    (4096, 9216, 16, 7, {(1, 1): 100.6, (1, 2): 105.1, (1, 3): 104.7, (1, 4): 108.2, (1, 5): 105.2, (1, 6): 116.4, (1, 8): 117.7, (1, 10): 126.3, (1, 12): 126.6, (1, 16): 136.9}, 105.6),
    (4096, 4096, 16, 18, {(1, 1): 121.2, (1, 2): 124.0, (1, 3): 127.4, (1, 4): 123.1, (1, 5): 125.5, (1, 6): 134.1, (1, 8): 135.6, (1, 10): 142.4, (1, 12): 143.1, (1, 16): 154.7}, 118.6),
    (4608, 2048, 256, 1, {(1, 2): 19.9, (1, 3): 17.6, (1, 4): 17.2, (1, 5): 18.5, (1, 6): 17.2, (1, 8): 17.8, (1, 12): 19.9, (2, 4): 19.4, (2, 5): 17.8, (2, 6): 17.1, (2, 8): 17.6, (3, 5): 20.1, (3, 6): 19.5, (3, 8): 19.8}, 36.0),
    (4608, 2048, 16, 7, {(1, 1): 27.4, (1, 2): 27.6, (1, 3): 28.4, (1, 4): 27.4, (1, 5): 30.6, (1, 6): 29.4, (1, 8): 28.6, (1, 10): 31.5, (1, 12): 31.3, (1, 16): 33.1}, 29.5),
    (2048, 4608, 128, 8, {(1, 1): 66.6, (1, 2): 74.6, (1, 3): 79.2, (1, 4): 78.4, (1, 5): 86.4, (1, 6): 99.7, (1, 8): 110.5, (2, 1): 76.2, (2, 2): 71.4, (2, 3): 79.4, (2, 4): 87.3, (2, 5): 88.0, (2, 6): 89.7, (2, 8): 107.9}, 90.9),
]


def test_choices_against_measured_times(ask):
    for (K, N, r, g, times, before), choice in zip(MEASURED, ask([m[:4] + (SCRATCH,) for m in MEASURED])):
        assert times[choice] <= 1.26 * min(times.values()), (K, N, r, g, choice)
        assert times[choice] <= 1.06 * before, (K, N, r, g, choice)
