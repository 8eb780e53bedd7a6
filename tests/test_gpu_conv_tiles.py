"""Convolutions in tiles of 256 positions x 96 columns, bf16, against the CPU oracle: columns that fill one or two tiles and that do
not, forward and input gradient, rows too long for the patch of 256 positions (128 then), and a strided first layer with as many
tiles as the chip has compute units and with fewer.  No ReLU and no max-pooling: a sign or a winner that rounding decides moves
single elements by as much as they are.  Every call is large enough to be served layer by layer."""
import pytest

from test_gpu_net import check_gradient, one_gradient

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def net(c, h, w, *layers):
    return {"name": "tiles", "input": (c, h, w), "classes": 8, "layers": list(layers) + [("fc", 24), ("fc", 8)]}


CASES = {
    # name: (network, mini-batch size, learners)
    "columns_96": (net(3, 12, 12, ("conv", 96, 3, 1, 1), ("conv", 160, 5, 1, 2), ("avgpool", 3, 2), ("conv", 96, 3, 1, 1)), 5, 3),
    "columns_72": (net(3, 9, 11, ("conv", 72, 3, 1, 1), ("conv", 96, 2, 1, 0), ("conv", 72, 3, 1, 1)), 4, 64),
    "columns_192": (net(3, 13, 13, ("conv", 192, 3, 1, 1), ("conv", 64, 3, 1, 1), ("avgpool", 3, 2), ("conv", 168, 3, 1, 1)), 4, 16),
    "columns_280": (net(3, 7, 7, ("conv", 280, 3, 1, 1), ("conv", 32, 3, 1, 0), ("conv", 280, 3, 1, 1)), 6, 64),
    "long_rows": (net(3, 6, 100, ("conv", 96, 3, 1, 1), ("conv", 32, 3, 1, 1), ("conv", 96, 3, 1, 1), ("avgpool", 3, 2)), 3, 8),
    "strided_first_full": (net(3, 47, 47, ("conv", 96, 11, 4, 0), ("avgpool", 3, 2)), 8, 64),
    "strided_first_few": (net(3, 47, 47, ("conv", 96, 11, 4, 0), ("avgpool", 3, 2)), 32, 8),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_convolution(name):
    nt, mu, lam = CASES[name]
    for (g, rg, loss, rl) in one_gradient(nt, mu, "bf16", seed=sum(map(ord, name)), scale=0.1, lam=lam):
        check_gradient(nt, "bf16", g, rg, loss, rl, name)
