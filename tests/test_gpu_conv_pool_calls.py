"""Which calls take the kernel of a first convolution and the max pooling behind it: the rule, compiled for the host, and a context whose calls fall on both
sides of it, against the CPU oracle."""
import os
import subprocess

import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
from oracle import cnn                                            # noqa: E402
from test_gpu_net import check_gradient, draw_case                # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "tile_rules.hpp"
int main() {
  int images, positions, C, Ncols, ks;
  while (scanf("%d %d %d %d %d", &images, &positions, &C, &Ncols, &ks) == 5) printf("%d\n", (int)sasgd::conv_pool_wins(images, positions, C, Ncols, ks));
}
"""
# Measured, us: images, positions, input channels, filters, window; separate kernels, one kernel
MEASURED = [
    (1024, 42, 16, 96, 3, 20.1, 17.9), (2048, 42, 16, 96, 3, 23.6, 30.7), (4096, 42, 16, 96, 3, 33.1, 59.0), (4096, 70, 32, 128, 2, 49.7, 69.6),
    (4096, 99, 8, 64, 2, 37.3, 33.3), (7680, 289, 64, 8, 2, 119.8, 150.6), (7680, 324, 64, 64, 5, 552.3, 608.6), (2048, 1280, 64, 16, 3, 220.2, 181.6),
    (2048, 324, 48, 32, 5, 100.0, 89.2), (7680, 576, 8, 16, 5, 145.3, 102.2), (1024, 576, 112, 8, 1, 40.1, 36.2), (256, 2916, 48, 96, 3, 149.0, 113.0),
]


def test_the_rule_takes_the_faster_way(tmp_path):
    (tmp_path / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(tmp_path / "rule.cpp"), "-o", str(tmp_path / "rule")], check=True)
    out = subprocess.run([str(tmp_path / "rule")], input="\n".join(" ".join(map(str, m[:5])) for m in MEASURED), capture_output=True, text=True, check=True).stdout
    assert [line == "1" for line in out.split()] == [m[6] < m[5] for m in MEASURED]


@pytest.mark.gpu
def test_calls_on_both_sides():
    """34 learners x 32 images of 7 x 9 positions go through separate kernels, 20 of them through one, in one context and both ways round."""
    from paper_1511_05950_amd import binding
    nt = {"name": "pool", "input": (3, 7, 9), "classes": 16, "layers": [("conv", 64, 5, 1, 2), ("maxpool", 3, 2), ("relu",), ("fc", 136), ("fc", 16)]}
    lam, mu = 34, 32
    theta, X, Y = draw_case(nt, lam, mu, 5, 0.1)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    want = {k: cnn.loss_and_gradient(nt, theta, X[k * mu:(k + 1) * mu], Y[k * mu:(k + 1) * mu], round_bf16=True) for k in (0, 19)}
    ctx = binding.Sasgd(lam, mu, lam, 2, net=nt, compute="bf16", init_weights=theta)
    loss = torch.zeros(lam, device="cuda")
    for count in (lam, 20, lam):
        for k in range(count):
            ctx.getMinibatch(k, Xd[k * mu:(k + 1) * mu], Yd[k * mu:(k + 1) * mu])
            ctx.pullWeights(k, 0)
        ctx.calcGradient(list(range(count)), loss)
        for k, (rl, rg) in want.items():
            check_gradient(nt, "bf16", ctx.copyGradient(k), rg, float(loss[k].item()), rl, str(count))
    ctx.destroy()
