"""Layers whose index arithmetic leaves 32 bits: more output positions than a 32-bit multiplier divides by the row length, and fully
connected layers of several hundred thousand inputs."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_net import check_gradient, one_gradient, rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

POSITIONS = {"name": "positions", "input": (3, 512, 512), "classes": 10,
             "layers": [("conv", 8, 3, 1, 1), ("avgpool", 8, 8), ("avgpool", 8, 8), ("fc", 10)]}


@pytest.mark.parametrize("compute", ["fp32", "bf16"])
def test_many_positions(compute):
    """33 images of 512 x 512, all zero but the last: positions x row length goes beyond 2^32 inside that one.  Its part of the first
    filter's gradient is a 33rd of what it is alone."""
    from paper_1511_05950_amd import binding
    theta = (np.random.default_rng(2).standard_normal(wl.num_params(POSITIONS)) * 0.1).astype(np.float32)
    theta[wl.num_params(POSITIONS) - 10:] = 0
    theta[8 * 27:8 * 28] = 0                                      # no bias: a zero image has zero scores and zero filter gradient
    image = torch.randn((1, 3, 512, 512), device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    out = []
    for mu in (1, 33):
        x = torch.zeros((mu, 3, 512, 512), device="cuda")
        x[-1] = image[0]
        y = torch.full((mu,), 4, dtype=torch.int32, device="cuda")
        ctx = binding.Sasgd(1, mu, 1, 1, net=POSITIONS, compute=compute, init_weights=theta)
        ctx.getMinibatch(0, x, y)
        ctx.pullWeights(0)
        ctx.calcGradient([0])
        out.append(mu * ctx.copyGradient(0)[:8 * 27].astype(np.float64))
        ctx.destroy()
    # a column of 512 left out is one part in 22 of a sum of random signs; 33 is no power of two, so bf16 rounds differently
    assert rel(out[1], out[0]) < (1e-4 if compute == "fp32" else 1e-2)


@pytest.mark.parametrize("compute, shape, mu", [("fp32", (3, 320, 320), 2), ("bf16", (8, 260, 260), 2), ("bf16", (8, 260, 260), 40)])
def test_many_inputs(compute, shape, mu):
    net = {"name": "inputs", "input": shape, "classes": 4, "layers": [("fc", 8), ("fc", 4)]}
    for (g, rg, loss, rl) in one_gradient(net, mu, compute, seed=6, scale=0.002, lam=1):
        check_gradient(net, compute, g, rg, loss, rl, "many inputs")


def test_inputs_that_fit_but_for_the_factors_rounding():
    """249 images of 2 144 000 inputs: their tensors stay below 2 GiB in 32 bits, and those of rows rounded up to 256 would not.  The layer then
    keeps no factors."""
    from paper_1511_05950_amd import binding
    net = {"name": "inputs", "input": (8, 500, 536), "classes": 4, "layers": [("fc", 8), ("fc", 4)]}
    assert 249 * 2_144_000 * 4 < 2 ** 31 < 256 * 2_144_000 * 4
    ctx = binding.Sasgd(1, 249, 1, 1, net=net, compute="bf16", init_weights=torch.zeros(wl.num_params(net), device="cuda"))
    assert ctx.factoredParams() == 0
    ctx.destroy()
