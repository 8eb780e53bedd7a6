"""How often a fully connected layer's product is split (csrc/tile_rules.hpp, compiled for the host), at long and at short contractions."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "tile_rules.hpp"
int main() {
  int K, N, rows, groups;
  while (scanf("%d %d %d %d", &K, &N, &rows, &groups) == 4) {
    const sasgd::FcRowsChoice c = sasgd::fc_rows_choice(K, N, rows, groups, 128 << 20);
    printf("%d %d\n", c.tm, c.splits);
  }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)

    def run(queries):
        out = subprocess.run([str(d / "rule")], input="\n".join(" ".join(map(str, q)) for q in queries), capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def test_splits_are_valid_for_long_contractions(ask):
    """Beyond 9 728 inputs: no workgroup without a stage, nine stages each at the least, and the partial sums have room."""
    queries = [(K, N, rows, g) for K in (9736, 19600, 65536, 416752, 8_000_000) for N in (8, 104, 1000) for rows in (1, 40, 300, 4096) for g in (1, 19, 64)]
    for (K, N, rows, g), (tm, sp) in zip(queries, ask(queries)):
        stages = -(-K // 64)
        per = -(-stages // sp)
        assert 1 <= sp <= 128 and -(-stages // per) == sp and (sp <= 16 or per >= 9)
        assert sp == 1 or (sp * rows * N * 4 <= 128 << 20 and rows * N * 4 < 2 ** 31)


def test_short_contractions_are_not_split(ask):
    queries = [(K, N, rows, g) for K in (8, 512, 1088) for N in (8, 1000, 9216) for rows in (1, 40, 300) for g in (1, 7)]
    assert all(sp == 1 for _, sp in ask(queries))


def test_few_columns_of_long_contractions_fill_the_chip(ask):
    """One tile of columns, few rows: 16 workgroups were all that such a product had."""
    for (K, N, rows), (_, sp) in zip([(161280, 88, 24), (349272, 24, 33), (81536, 112, 11)], ask([(161280, 88, 24, 1), (349272, 24, 33, 1), (81536, 112, 11, 1)])):
        assert sp >= 96, (K, N, rows)
