"""Fully connected layers, bf16, against the CPU oracle: from one row to 2 048 rows of one weight version, every height of tile, contractions
split and not, rows, columns and contractions that end inside a tile.  No ReLU and no max-pooling (test_gpu_net.py has those): a sign
that rounding decides moves single elements by as much as they are."""
import pytest

from test_gpu_net import check_gradient, one_gradient

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WIDE = {"name": "rows", "input": (3, 12, 12), "classes": 24,                  # 1 152 -> 3 080 -> 24
        "layers": [("conv", 32, 3, 1, 1), ("avgpool", 3, 2), ("fc", 3080), ("fc", 24)]}
SMALL = {"name": "rows", "input": (3, 6, 6), "classes": 16,                   # 72 -> 200 -> 16
         "layers": [("conv", 8, 3, 1, 1), ("avgpool", 3, 2), ("fc", 200), ("fc", 16)]}

CASES = {
    # name: (network, mini-batch size, learners, (heights of a tile in 64 rows, split or not) of the layer behind the convolution, both ways)
    "one_row": (WIDE, 1, 1, ((1, True), (1, True))),
    "rows_34": (WIDE, 17, 2, ((1, True), (1, True))),
    "rows_65": (WIDE, 13, 5, ((1, True), (1, True))),
    "rows_192": (WIDE, 32, 6, ((1, False), (1, True))),
    "rows_767": (WIDE, 13, 59, ((2, False), (1, True))),
    "rows_1536": (WIDE, 32, 48, ((3, False), (1, False))),
    "rows_1920": (WIDE, 30, 64, ((3, False), (3, True))),
    "rows_2048": (WIDE, 32, 64, ((4, False), (2, False))),
    "small_21": (SMALL, 7, 3, ((1, False), (1, False))),
    "small_320": (SMALL, 32, 10, ((1, False), (1, False))),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_layers(name):
    nt, mu, lam, _ = CASES[name]
    seed = sum(map(ord, name))
    for (g, rg, loss, rl) in one_gradient(nt, mu, "bf16", seed=seed, scale=0.05, lam=lam, learners=sorted({0, lam // 2, lam - 1})):
        check_gradient(nt, "bf16", g, rg, loss, rl, name)
