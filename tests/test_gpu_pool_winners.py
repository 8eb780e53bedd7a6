"""Max-pooling behind a ReLU, layer by layer, against the CPU oracle: windows whose maximum is not positive, which no gradient passes,
in every kernel that keeps and reads winners: 3 x 3 at stride 2, other windows from 1 x 1 (half of them without a positive value) to
the largest, channels that are no multiple of 8, fp32; images in a space-to-depth first layer whose last row of pixels is cut.
Enough learners that a call is not small.  One ReLU and one max-pooling a network, on sums of a few hundred terms at most: in bf16 few of
their decisions differ from the reduced-precision oracle's, in fp32 none does (decided_seed)."""
import pytest

from test_gpu_net import check_gradient, decided_seed, one_gradient

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

R = ("relu",)


def net(h, w, *layers):
    return {"name": "winners", "input": (3, h, w), "classes": 8, "layers": list(layers) + [("fc", 24), ("fc", 8)]}


CASES = {
    # name: (network, compute, mini-batch size, learners)
    "pool_3_2": (net(13, 11, ("conv", 16, 3, 1, 1), R, ("maxpool", 3, 2)), "bf16", 2, 64),
    "pool_3_1": (net(9, 10, ("conv", 16, 3, 1, 1), R, ("maxpool", 3, 1)), "bf16", 2, 64),
    "pool_2_2": (net(11, 9, ("conv", 24, 3, 1, 1), R, ("maxpool", 2, 2)), "bf16", 2, 64),
    "pool_1_1": (net(7, 9, ("conv", 16, 3, 1, 1), R, ("maxpool", 1, 1)), "bf16", 2, 64),
    "pool_15_4": (net(22, 19, ("conv", 16, 3, 1, 1), R, ("maxpool", 15, 4)), "bf16", 2, 64),
    "odd_channels": (net(11, 9, ("conv", 13, 3, 1, 1), R, ("maxpool", 2, 2)), "bf16", 2, 64),
    "cut_row": (net(45, 48, ("conv", 16, 11, 4, 0), R, ("maxpool", 2, 2)), "bf16", 2, 64),
    # (windows that overlap by more than half: no small-call kernel takes them)
    "fp32": (net(16, 16, ("conv", 8, 3, 1, 1), R, ("maxpool", 3, 1), ("conv", 16, 3, 1, 1)), "fp32", 4, 4),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_gradient_below_max_pooling(name):
    nt, compute, mu, lam = CASES[name]
    seed = sum(map(ord, name))
    if compute == "fp32":
        seed = decided_seed(nt, lam, mu, seed, 0.1)
    for (g, rg, loss, rl) in one_gradient(nt, mu, compute, seed=seed, scale=0.1, lam=lam):
        check_gradient(nt, compute, g, rg, loss, rl, name)
