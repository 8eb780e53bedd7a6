"""Flattening in front of a fully connected layer: the rule by which a call's kernel is chosen, compiled for the host, and both kernels and every form of the
tiles against the CPU oracle: maps that end inside a tile of 64 positions and that fill it, blocks of 64 channels whole and cut, whole 16-byte pieces on
each side and none, one image and many."""
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
  long images;
  int C, HW, bf16;
  while (scanf("%ld %d %d %d", &images, &C, &HW, &bf16) == 4) {
    const sasgd::FlattenPlan p = sasgd::flatten_plan(images, C, HW, bf16 != 0);
    printf("%d %d %d %ld\n", (int)p.direct, (int)p.pieces, p.rows, (long)p.groups);
  }
}
"""
DIRECT, ELEMENTS, PIECES, BLOCK, BLOCK_128 = -1, 0, 1, 2, 3
# height, width, channels, window of the convolution, hidden units, learners, images of each, the positions' side of the tiles: what keeps a call layer by
# layer (in bf16 a hidden layer whose factors are kept, or a large one behind channels that are no multiple of 8)
CASES = [
    (13, 10, 64, 3, 16, 64, 4, ELEMENTS),        # 130 positions
    (16, 8, 72, 3, 16, 64, 4, PIECES),           # 128 positions, 64 + 8 channels
    (9, 7, 136, 3, 16, 64, 4, BLOCK),            # 63 positions
    (8, 8, 64, 3, 16, 64, 4, BLOCK),             # a full tile
    (13, 5, 64, 3, 16, 64, 4, BLOCK_128),        # 65 positions
    (1, 127, 72, 3, 16, 64, 4, BLOCK_128),
    (10, 20, 44, 1, 512, 64, 24, PIECES),        # single channels
    (11, 14, 68, 1, 512, 64, 24, ELEMENTS),      # single channels beyond a block
    (31, 33, 8, 3, 16, 64, 2, DIRECT),           # few channels, single positions
    (32, 32, 8, 3, 16, 64, 2, PIECES),
    (17, 15, 24, 3, 16, 3, 2, DIRECT),           # few values
    (45, 45, 16, 3, 16, 1, 1, DIRECT),
]
# fp32: two convolutions of some size
CASES32 = [(13, 10, 64, 64, 24, ELEMENTS), (16, 8, 72, 64, 16, PIECES), (9, 7, 68, 64, 24, BLOCK), (13, 5, 64, 64, 24, BLOCK_128), (31, 33, 4, 64, 8, DIRECT),
           (13, 10, 64, 1, 40, DIRECT)]


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)

    def run(queries):
        out = subprocess.run([str(d / "rule")], input="\n".join(" ".join(map(str, q)) for q in queries), capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def test_every_call_has_workgroups_for_its_values(ask):
    queries = [(n, C, hw, bf) for n in (1, 16, 576) for C in (1, 8, 10, 43, 64, 72, 256) for hw in (4, 25, 256, 625, 1024, 10000) for bf in (0, 1)]
    for (n, C, hw, bf), (direct, pieces, rows, groups) in zip(queries, ask(queries)):
        assert groups * (256 if direct else 64 * (128 if rows == BLOCK_128 else 64)) >= C * hw
        assert groups >= -(-C * hw // 4096)               # one image of 64 x 32 x 32 on 16 workgroups at the least
        assert rows < BLOCK or (pieces and hw <= 64 * (rows - 1))
        assert rows != PIECES or hw % (8 if bf else 4) == 0
        assert not pieces or C % (8 if bf else 4) == 0


def test_the_gpu_cases_reach_every_form(ask):
    for cases, bf, seen in ((CASES, 1, {(1, ELEMENTS), (0, ELEMENTS), (1, PIECES), (0, PIECES), (1, BLOCK), (1, BLOCK_128)}),
                            (CASES32, 0, {(1, ELEMENTS), (1, PIECES), (1, BLOCK), (1, BLOCK_128)})):
        got = ask([(k[-3] * k[-2], k[2], k[0] * k[1], bf) for k in cases])
        assert [DIRECT if d else rows for d, _, rows, _ in got] == [k[-1] for k in cases]
        assert seen == {(pieces, rows) for d, pieces, rows, _ in got if not d}


@pytest.mark.gpu
@pytest.mark.parametrize("h, w, c, ks, hidden, lam, mu, form", CASES)
def test_flatten_bf16(h, w, c, ks, hidden, lam, mu, form):
    nt = {"name": "flat", "input": (3, h, w), "classes": 8, "layers": [("conv", c, ks, 1, ks // 2), ("relu",), ("fc", hidden), ("fc", 8)]}
    for (g, rg, loss, rl) in one_gradient(nt, mu, "bf16", seed=11 * h + c, scale=0.1, lam=lam, learners=sorted({0, lam - 1})):
        check_gradient(nt, "bf16", g, rg, loss, rl, "flatten")


@pytest.mark.gpu
@pytest.mark.parametrize("h, w, c, lam, mu, form", CASES32)
def test_flatten_fp32(h, w, c, lam, mu, form):
    nt = {"name": "flat", "input": (3, h, w), "classes": 8, "layers": [("conv", 64, 5, 1, 2), ("conv", c, 5, 1, 2), ("fc", 8)]}
    for (g, rg, loss, rl) in one_gradient(nt, mu, "fp32", seed=11 * h + c, scale=0.1, lam=lam, learners=sorted({0, lam - 1})):
        check_gradient(nt, "fp32", g, rg, loss, rl, "flatten")
