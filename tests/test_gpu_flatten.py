"""Flattening in front of a fully connected layer and its backward pass, layer by layer, against the CPU oracle: channels that fill blocks of 64 and
that do not, in whole 16-byte pieces and not, images whose tile fits LDS and one whose tile does not."""
import pytest

from test_gpu_net import check_gradient, decided_seed, one_gradient

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def net(h, w, c):
    return {"name": "flat", "input": (3, h, w), "classes": 8, "layers": [("conv", c, 3, 1, 1), ("fc", 8)]}


@pytest.mark.parametrize("compute", ["fp32", "bf16"])
@pytest.mark.parametrize("h, w, c", [(7, 9, 72), (5, 5, 136), (6, 7, 64), (24, 23, 8), (6, 5, 68)])
def test_flatten(compute, h, w, c):
    nt = net(h, w, c)
    seed = 11 * h + c if compute == "bf16" else decided_seed(nt, 64, 8, 11 * h + c, 0.1)
    for (g, rg, loss, rl) in one_gradient(nt, 8, compute, seed=seed, scale=0.1, lam=64, learners=[0, 63]):
        check_gradient(nt, compute, g, rg, loss, rl, "flatten")
