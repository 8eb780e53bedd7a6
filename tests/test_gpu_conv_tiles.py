"""Convolutions of more than 64 columns, bf16, against the CPU oracle, forward and input gradient: tiles of 256 positions x 96 columns, of
256 x 128 and of 128 x 128, columns that fill one or two tiles and that do not, contractions split and not, rows too long for the patch
of 256 positions, channels that are no multiple of 32 (tap by tap) and a strided first layer.  No ReLU and no max-pooling: a sign
or a winner that rounding decides moves single elements by as much as they are.  Every call is large enough to be served layer by
layer."""
import pytest

from test_gpu_net import bounded_learners, check_gradient, one_gradient

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
    # calls that fill the chip with the larger tiles
    "tiles_96": (net(3, 11, 12, ("conv", 96, 3, 1, 1), ("conv", 160, 2, 1, 0), ("conv", 96, 3, 1, 1), ("avgpool", 3, 2)), 6, 48),
    "tiles_72": (net(3, 13, 13, ("conv", 64, 3, 1, 1), ("conv", 72, 3, 1, 1), ("conv", 72, 3, 1, 1), ("avgpool", 3, 2)), 8, 12),
    "tiles_192": (net(3, 9, 9, ("conv", 192, 3, 1, 1), ("conv", 64, 3, 1, 1), ("conv", 168, 3, 1, 1), ("avgpool", 3, 2)), 8, 24),
    "tiles_280": (net(3, 9, 9, ("conv", 280, 3, 1, 1), ("conv", 32, 3, 1, 1), ("conv", 280, 3, 1, 1), ("avgpool", 3, 2)), 8, 48),
    "tiles_384": (net(3, 9, 9, ("conv", 384, 3, 1, 1), ("conv", 96, 3, 1, 1), ("conv", 384, 3, 1, 1), ("avgpool", 3, 2)), 8, 48),
    "tiles_long_rows": (net(3, 6, 100, ("conv", 96, 3, 1, 1), ("conv", 32, 3, 1, 1), ("conv", 96, 3, 1, 1), ("avgpool", 3, 2)), 4, 48),
    "tiles_strided_first": (net(3, 47, 47, ("conv", 96, 11, 4, 0), ("avgpool", 3, 2)), 12, 12),
}

# the tiles that these take, forward passes first to last, then input gradients (asked of the rules, without a GPU)
REACHES = {
    "tiles_96": ("256x96",) * 4, "tiles_72": ("256x96", "taps 256x96", "taps 256x96"), "tiles_192": ("256x96",) * 2, "tiles_280": ("256x96",) * 2,
    "tiles_384": ("256x96 split", "256x128") * 2, "tiles_long_rows": ("256x96",) * 2, "tiles_strided_first": ("taps 256x96",),
    "columns_96": ("128x128 split",) * 4,
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_convolution(name):
    nt, mu, lam = CASES[name]
    seed = sum(map(ord, name))
    # every learner's gradient, or the first one's, one's in the middle and the last one's
    learners = range(lam) if not name.startswith("tiles") else bounded_learners(nt, lam, mu, seed, 0.1, sorted({0, lam // 2, lam - 1}))
    for (g, rg, loss, rl) in one_gradient(nt, mu, "bf16", seed=seed, scale=0.1, lam=lam, learners=learners):
        check_gradient(nt, "bf16", g, rg, loss, rl, name)
