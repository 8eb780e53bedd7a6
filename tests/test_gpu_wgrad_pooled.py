"""A first convolution's weight gradient that takes the gradient of the 3 x 3 / 2 max pooling's output behind it, against the same layers with the
pooling layer's backward kernel in between, bit by bit: every form of the kernel, even images whose tiles end in a row of another image or
beyond the last one, windows that the image cuts, channels that fill no block, and layers just outside the rule."""
import os
import subprocess

import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
from test_gpu_net import draw_case            # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
R, P, F = ("relu",), ("maxpool", 3, 2), ("fc", 16)
# name: image, convolution, mini-batch, learners, the kernel's form (-1: one that reads its own output's gradient)
CASES = {
    "few_columns": ((8, 32, 32), (32, 5, 1, 2), 9, 8, 2),
    "few_columns_24_filters": ((8, 18, 16), (24, 5, 1, 2), 15, 16, 2),
    "few_columns_rows_of_64": ((8, 14, 64), (16, 3, 1, 1), 10, 8, 2),
    "few_columns_no_padding": ((8, 36, 36), (32, 5, 1, 0), 8, 8, 2),
    "few_columns_40_filters": ((8, 20, 32), (40, 5, 1, 2), 13, 8, 0),
    "few_columns_rows_of_8": ((8, 30, 8), (64, 3, 1, 1), 35, 8, 0),
    "columns_64_filters": ((16, 22, 16), (64, 5, 1, 2), 13, 16, 1),
    "columns_32_filters": ((16, 22, 16), (32, 5, 1, 2), 13, 16, 3),
    "many_columns": ((32, 16, 16), (24, 5, 1, 2), 17, 16, 4),
    "odd_rows": ((8, 31, 32), (32, 5, 1, 2), 9, 8, -1),
    "tiles_of_no_whole_rows": ((8, 24, 24), (32, 5, 1, 2), 15, 8, -1),
}
PROGRAM = r"""
#include <stdio.h>
#include "tile_rules.hpp"
int main() {
  sasgd::StripLayer g;
  sasgd::StripPlan p;
  if (scanf("%d %d %d %d %d %d %d %d %d", &g.M, &g.Ncols, &g.C, &g.ks, &g.OH, &g.OW, &g.W, &g.pad, &g.count) != 9) return 1;
  g.scratch_bytes = 128 << 20;
  printf("%d\n", sasgd::strip_plan(g, &p) && sasgd::strip_pools(p, g.OH, g.OW) ? p.form : -1);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)
    return str(d / "rule")


@pytest.mark.parametrize("name", sorted(CASES))
def test_forms(rule, name):
    (c, h, w), (k, ks, _, pad), mu, lam, form = CASES[name]
    oh, ow = h + 2 * pad - ks + 1, w + 2 * pad - ks + 1
    got = subprocess.run([rule], input=" ".join(map(str, (mu * oh * ow, k, c, ks, oh, ow, w, pad, lam))), capture_output=True, text=True, check=True)
    assert int(got.stdout) == form


@pytest.mark.parametrize("tm,mt", [(2, 256), (1, 512), (1, 256)])
def test_threads_cover_a_tile(tm, mt):
    """The threads' 2 x 2 blocks are a tile's positions, each once, and every window that covers a position is one of its block's four."""
    for ow in [2 ** k for k in range(1, 9) if mt % 2 ** (k + 1) == 0]:
        seen = set()
        for tid in range(tm * mt):
            chunk, block = tid % (tm * 4), tid // (tm * 4)
            row = 2 * block // ow
            col = block - row * (ow // 2)
            for q in range(4):
                r, c = 2 * row + q // 2, 2 * col + q % 2
                seen.add((chunk, r * ow + c))
                windows = {(a, b) for a in range(-1, r + 1) for b in range(col - 2, c + 1) if 0 <= r - 2 * a <= 2 and 0 <= c - 2 * b <= 2}
                assert windows <= {(row + a, col + b) for a in (-1, 0) for b in (-1, 0)}
        assert len(seen) == tm * 4 * mt and max(p for _, p in seen) == mt - 1


BLOCKS = r"""
#include <stdio.h>
#include "tile_rules.hpp"
int main() {
  int tm, mt, ow;
  if (scanf("%d %d %d", &tm, &mt, &ow) != 3) return 1;
  for (int tid = 0; tid < tm * mt; tid++) {
    const sasgd::PoolBlock b = sasgd::pool_block(tid, tm, ow, [&](uint32_t n) { return n / (uint32_t)ow; });
    printf("%d %d %d %d\n", b.chunk, b.row, b.col, b.first);
  }
}
"""


def test_the_kernels_blocks_cover_a_tile(tmp_path):
    """As above, of the function that places the kernel's threads."""
    (tmp_path / "blocks.cpp").write_text(BLOCKS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(tmp_path / "blocks.cpp"), "-o", str(tmp_path / "blocks")], check=True)
    for tm, mt in [(2, 256), (1, 512), (1, 256)]:
        for ow in [k for k in range(2, mt // 2 + 1, 2) if mt % (2 * k) == 0]:
            out = subprocess.run([str(tmp_path / "blocks")], input="%d %d %d" % (tm, mt, ow), capture_output=True, text=True, check=True).stdout
            seen = set()
            for chunk, row, col, first in (map(int, line.split()) for line in out.splitlines()):
                for q in range(4):
                    p = first + q // 2 * ow + q % 2
                    seen.add((chunk, p))
                    r, c = divmod(p, ow)
                    windows = {(a, b) for a in range(-1, r + 1) for b in range(-1, c + 1) if 0 <= r - 2 * a <= 2 and 0 <= c - 2 * b <= 2}
                    assert windows <= {(row + a, col + b) for a in (-1, 0) for b in (-1, 0)}
            assert seen == {(chunk, p) for chunk in range(tm * 4) for p in range(mt)}


@pytest.mark.gpu
@pytest.mark.parametrize("relu_first", [True, False])
@pytest.mark.parametrize("name", sorted(CASES))
def test_same_bits_as_through_the_pooling_layer(name, relu_first):
    """Images of bf16 values behind a 1 x 1 convolution that copies them: the layer is the second one there, which needs its output's gradient
    for the input gradient too."""
    from paper_1511_05950_amd import binding
    (c, h, w), (k, ks, st, pad), mu, lam, _ = CASES[name]
    tail = [("conv", k, ks, st, pad)] + ([R, P] if relu_first else [P, R]) + [F]
    one = {"name": "pooled", "input": (c, h, w), "classes": 16, "layers": tail}
    two = {"name": "pooled", "input": (c, h, w), "classes": 16, "layers": [("conv", c, 1, 1, 0)] + tail}
    theta, X, Y = draw_case(one, lam, mu, sum(map(ord, name)), 0.05)
    X = torch.from_numpy(X).cuda().bfloat16().float()
    Yd = torch.from_numpy(Y).cuda()
    copy = np.concatenate([np.eye(c, dtype=np.float32).ravel(), np.zeros(c, np.float32), theta])
    got = []
    for nt, start in ((one, theta), (two, copy)):
        ctx = binding.Sasgd(lam, mu, lam, 2, net=nt, compute="bf16", init_weights=start)
        loss = torch.zeros(lam, device="cuda")
        for _ in range(2):                     # the second pass finds the first one's values in the workspace
            for j in range(lam):
                ctx.pullWeights(j, 0)
                ctx.getMinibatch(j, X[j * mu:(j + 1) * mu], Yd[j * mu:(j + 1) * mu])
            ctx.calcGradient(list(range(lam)), loss)
        got.append([loss.cpu().numpy()] + [ctx.copyGradient(j)[-wl.num_params(one):] for j in range(lam)])
        ctx.destroy()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    assert np.abs(got[0][1][:k * c * ks * ks]).max() > 0
