"""Fully connected layers, bf16, in the forms for few rows and for short contractions, against the CPU oracle: forward products without LDS, tiles of 32
rows, one and two stages in every height of tile with the ReLU mask beside the operands, and more than sixteen splits; rows, columns and
contractions that end inside what a workgroup takes.  The rules are compiled for the host."""
import os
import subprocess

import pytest

pytest.importorskip("torch")
from test_gpu_net import check_gradient, one_gradient            # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "tile_rules.hpp"
int main() {
  int K, N, rows, groups;
  while (scanf("%d %d %d %d", &K, &N, &rows, &groups) == 4) {
    const sasgd::FcRowsChoice c = sasgd::fc_rows_choice(K, N, rows, groups, 128 << 20);
    printf("%d %d %d\n", (int)sasgd::fc_rows_short(K, N, rows, groups), c.tm, c.splits);
  }
}
"""
# name: height and width behind 8 filters, hidden units, images, learners, form of the hidden layer's forward product and of its input gradient:
# "short", or (tile of 32 rows: 0, else its height in 64 rows; stages in LDS)
CASES = {
    "one_row": (5, 5, 72, 1, 1, "short", (0, 2)),
    "few_rows": (1, 3, 200, 3, 7, "short", (0, 3)),
    "rows_32": (16, 16, 264, 8, 4, "short", (0, 3)),
    "rows_30_of_10000": (25, 50, 24, 5, 6, (0, 3), (0, 1)),
    "rows_29": (25, 50, 104, 29, 1, (0, 3), (0, 2)),
    "rows_33": (5, 5, 72, 11, 3, (1, 3), (1, 2)),
    "rows_49": (25, 50, 24, 7, 7, (1, 3), (1, 1)),
    "rows_300_one_stage": (25, 50, 24, 20, 15, None, (2, 1)),
    "rows_300_two_stages": (25, 50, 104, 20, 15, None, (2, 2)),
    "rows_400_one_stage": (25, 50, 24, 20, 20, None, (3, 1)),
    "rows_400_two_stages": (25, 50, 104, 20, 20, None, (3, 2)),
    "rows_640_one_stage": (25, 50, 24, 32, 20, None, (4, 1)),
    "rows_640_two_stages": (25, 50, 104, 32, 20, None, (4, 2)),
    "forward_300_one_stage": (1, 3, 10000, 20, 15, (2, 1), None),
    "forward_300_two_stages": (3, 4, 10000, 20, 15, (2, 2), None),
    "forward_400_one_stage": (1, 3, 10000, 20, 20, (3, 1), None),
    "forward_400_two_stages": (3, 4, 10000, 20, 20, (3, 2), None),
    "forward_640_one_stage": (1, 3, 10000, 32, 20, (4, 1), None),
    "forward_640_two_stages": (3, 4, 10000, 32, 20, (4, 2), None),
    "many_splits": (60, 80, 16, 2, 3, (0, 3), (0, 1)),
}


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)

    def run(queries):
        out = subprocess.run([str(d / "rule")], input="\n".join(" ".join(map(str, q)) for q in queries), capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def form(K, rows, answer, forward):
    short, tm, splits = answer
    if forward and short:
        return "short"
    stages = -(-K // 64)
    return (0 if rows <= 32 else tm, min(3, -(-stages // splits)))


def test_the_gpu_cases_reach_the_forms(ask):
    for name, (h, w, hidden, mu, lam, fwd, back) in CASES.items():
        K, rows = 8 * h * w, mu * lam
        f, b = ask([(K, hidden, rows, 1), (hidden, K, rows, 1)])
        assert fwd is None or form(K, rows, f, True) == fwd, (name, f)
        assert back is None or form(hidden, rows, b, False) == back, (name, b)
    assert ask([(8 * 60 * 80, 16, 6, 1)])[0][2] > 16


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_layers(name):
    h, w, hidden, mu, lam, _, _ = CASES[name]
    nt = {"name": "rows", "input": (3, h, w), "classes": 16, "layers": [("conv", 8, 1, 1, 0), ("relu",), ("fc", hidden), ("relu",), ("fc", 16)]}
    for (g, rg, loss, rl) in one_gradient(nt, mu, "bf16", seed=sum(map(ord, name)), scale=0.1 if h * w < 1000 else 0.05, lam=lam, learners=sorted({0, lam - 1})):
        check_gradient(nt, "bf16", g, rg, loss, rl, name)
