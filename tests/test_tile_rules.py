"""The rules by which a call's kernels and tiles are chosen (csrc/tile_rules.hpp), compiled for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <string.h>
#include "tile_rules.hpp"
using namespace sasgd;
// stdin: a rule's name and its arguments; stdout: what it says, one line each
int main() {
  char rule[32];
  while (scanf("%31s", rule) == 1) {
    if (!strcmp(rule, "input")) {
      int bf16, s2d, C, Cp, Wp, aligned;
      if (scanf("%d %d %d %d %d %d", &bf16, &s2d, &C, &Cp, &Wp, &aligned) != 6) return 1;
      printf("%d %d\n", (int)input_layout(bf16, s2d, C, Cp, aligned), input_row_piece(Wp));
    } else if (!strcmp(rule, "pixels")) {
      int N, Hp, Wp;
      if (scanf("%d %d %d", &N, &Hp, &Wp) != 3) return 1;
      printf("%d\n", (int)input_pixel_groups(N, Hp, Wp));
    } else {
      return 1;
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    where = tmp_path_factory.mktemp("rules")
    src, exe = where / "rules.cpp", where / "rules"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(src), "-o", str(exe)])

    def run(questions):
        out = subprocess.check_output([str(exe)], input="\n".join(" ".join(map(str, q)) for q in questions), text=True).splitlines()
        assert len(out) == len(questions)
        return [tuple(float(x) if "." in x else int(x) for x in line.split()) for line in out]
    return run


def test_input_layout(ask):
    """Images of any width keep the row kernel, whose pieces of a row fit 60 KiB of LDS (96 bytes a pixel) and are even."""
    widths = [1, 56, 639, 640, 641, 768, 1280, 1281, 3000, 100_001]
    for wp, (layout, piece) in zip(widths, ask([("input", 1, 4, 3, 48, wp, 1) for wp in widths])):
        assert layout == 0 and 1 <= piece <= 640
        assert -(-wp // piece) == -(-wp // 640)
    assert [r[0] for r in ask([("input", 1, 4, 3, 48, 56, 0), ("input", 1, 2, 3, 16, 56, 1), ("input", 1, 1, 3, 8, 56, 1),
                               ("input", 0, 4, 3, 48, 56, 1), ("input", 1, 1, 13, 13, 56, 1)])] == [1, 1, 1, 2, 2]


def test_small_images_share_workgroups(ask):
    assert ask([("pixels", *q) for q in ((2048, 4, 4), (1, 3, 5), (4096, 3, 9), (128, 32, 32), (16, 512, 512))]) == [(128,), (1,), (432,), (512,), (16384,)]
