"""Weight gradients at the edges of the kernels' tiles, bf16, against the CPU
oracle: contractions of one and a few steps and of no whole number of them, image rows shorter and longer than a step, filter
taps that change inside a 32-column panel, the bias column alone in a tile, partly filled column tiles, splits of which the last one is
shorter, and a fully connected layer whose gradient is written out.  The networks hold no ReLU and no max-pooling: a sign or a winner that rounding decides
moves single elements by as much as they are, whichever way the sums are ordered."""
import pytest

import workloads as wl
from test_gpu_net import bounded_learners, check_gradient, one_gradient

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def net(c, h, w, *layers):
    return {"name": "tiles", "input": (c, h, w), "classes": 8, "layers": list(layers) + [("fc", 24), ("fc", 8)]}


CASES = {
    # name: (network, mini-batch size, learners)
    "one_step": (net(3, 5, 5, ("conv", 72, 3, 1, 0), ("conv", 136, 2, 1, 0)), 1, 1),
    "steps_2_to_4": (net(3, 8, 8, ("conv", 80, 3, 1, 0), ("conv", 72, 2, 1, 0)), 3, 2),
    "ragged": (net(3, 12, 11, ("conv", 128, 3, 1, 1), ("conv", 72, 3, 1, 1), ("avgpool", 3, 2), ("conv", 136, 5, 1, 2)), 3, 2),
    "wide_rows": (net(3, 9, 41, ("conv", 72, 3, 1, 1), ("conv", 96, 3, 1, 0), ("avgpool", 3, 2)), 2, 2),
    "stride_2": (net(3, 29, 27, ("conv", 80, 7, 2, 0), ("conv", 72, 3, 1, 0), ("avgpool", 3, 2)), 2, 2),
    "many_learners": (net(3, 8, 8, ("conv", 128, 3, 1, 1), ("conv", 256, 3, 1, 1), ("avgpool", 3, 2)), 4, 12),
    # the wide tiles (96 x 512, 256 x 256, 384 x 128), full and partly filled, one split: many learners make them the cheapest at few steps
    "wide_96": (net(3, 9, 9, ("conv", 224, 3, 1, 1), ("conv", 96, 3, 1, 1), ("avgpool", 3, 2)), 2, 64),
    "wide_88": (net(3, 7, 7, ("conv", 224, 3, 1, 1), ("conv", 88, 3, 1, 1), ("avgpool", 3, 2)), 3, 64),
    "wide_256": (net(3, 9, 9, ("conv", 112, 3, 1, 1), ("conv", 256, 3, 1, 1), ("avgpool", 3, 2)), 2, 64),
    "wide_200": (net(3, 9, 9, ("conv", 112, 3, 1, 1), ("conv", 200, 3, 1, 1), ("avgpool", 3, 2)), 2, 64),
    "wide_384": (net(3, 12, 11, ("conv", 40, 3, 1, 1), ("conv", 384, 3, 1, 1), ("avgpool", 3, 2)), 11, 64),
    "wide_360": (net(3, 13, 13, ("conv", 40, 3, 1, 1), ("conv", 360, 3, 1, 1), ("avgpool", 3, 2)), 8, 64),
    # several splits, the last one shorter, and a space-to-depth first layer
    "wide_96_splits": (net(3, 21, 23, ("conv", 56, 3, 1, 1), ("conv", 96, 3, 1, 1), ("avgpool", 3, 2)), 48, 16),
    "wide_88_splits": (net(3, 21, 23, ("conv", 48, 3, 1, 1), ("conv", 88, 3, 1, 1), ("avgpool", 3, 2)), 11, 64),
    "wide_256_splits": (net(3, 21, 23, ("conv", 24, 3, 1, 1), ("conv", 256, 3, 1, 1), ("avgpool", 3, 2)), 11, 64),
    "wide_200_splits": (net(3, 13, 13, ("conv", 24, 3, 1, 1), ("conv", 200, 3, 1, 1), ("avgpool", 3, 2)), 32, 64),
    "wide_384_splits": (net(3, 12, 11, ("conv", 24, 3, 1, 1), ("conv", 384, 3, 1, 1), ("avgpool", 3, 2)), 23, 48),
    "wide_360_splits": (net(3, 12, 11, ("conv", 16, 3, 1, 1), ("conv", 360, 3, 1, 1), ("avgpool", 3, 2)), 23, 48),
    "wide_strided_splits": (net(3, 71, 75, ("conv", 96, 11, 4, 0), ("avgpool", 3, 2)), 74, 18),
    # up to 64 output channels
    "narrow_one_step": (net(3, 5, 5, ("conv", 8, 3, 1, 0), ("conv", 64, 2, 1, 0)), 1, 1),
    "narrow_ragged": (net(3, 12, 11, ("conv", 32, 3, 1, 1), ("conv", 64, 5, 1, 2), ("avgpool", 3, 2), ("conv", 24, 3, 1, 1)), 5, 3),
    "narrow_wide_rows": (net(3, 9, 70, ("conv", 40, 3, 1, 1), ("conv", 32, 3, 1, 0), ("avgpool", 3, 2)), 2, 2),
    "narrow_full_tiles": (net(3, 16, 16, ("conv", 64, 3, 1, 1), ("conv", 32, 2, 1, 0), ("conv", 16, 4, 1, 1), ("avgpool", 3, 2)), 4, 12),
    # narrow layers of many positions: tiles inside an image, across lines, across many small images; one and several column groups
    "strip_first": (net(3, 32, 32, ("conv", 24, 5, 1, 2), ("avgpool", 3, 2)), 1, 64),
    "strip_ragged": (net(3, 31, 37, ("conv", 8, 4, 1, 0), ("conv", 32, 5, 1, 2), ("conv", 16, 3, 1, 1), ("avgpool", 3, 2)), 2, 64),
    "strip_small_images": (net(3, 9, 7, ("conv", 16, 3, 1, 1), ("conv", 24, 5, 1, 2), ("conv", 40, 3, 1, 1), ("avgpool", 3, 2)), 18, 64),
    "strip_two_rows": (net(3, 33, 32, ("conv", 32, 3, 1, 1), ("conv", 64, 3, 1, 1), ("avgpool", 3, 2)), 1, 64),
    "strip_no_padding": (net(3, 33, 32, ("conv", 32, 4, 1, 0), ("conv", 48, 3, 1, 0), ("avgpool", 3, 2)), 2, 64),
    "strip_groups": (net(3, 16, 16, ("conv", 32, 3, 1, 1), ("conv", 64, 5, 1, 2), ("conv", 32, 5, 1, 2), ("avgpool", 3, 2)), 4, 64),
    # space-to-depth first layers, whose second pass adds column by column: one split and a few, columns of one run of 256 and of several
    "strided_one_split": (net(3, 33, 35, ("conv", 40, 9, 2, 0), ("avgpool", 3, 2)), 1, 40),
    "strided_few_splits": (net(3, 47, 45, ("conv", 104, 11, 2, 0), ("avgpool", 3, 2)), 3, 12),
    "strided_many_splits": (net(3, 47, 45, ("conv", 24, 11, 4, 0), ("avgpool", 3, 2)), 48, 3),
    "most_splits": (net(3, 93, 91, ("conv", 72, 3, 1, 1), ("avgpool", 3, 2)), 12, 1),
    # many taps per channel, input channels in groups of which the last is shorter
    "many_taps": (net(3, 20, 20, ("conv", 40, 3, 1, 1), ("conv", 24, 11, 1, 5), ("avgpool", 3, 2)), 3, 2),
    "uneven_groups": (net(3, 12, 12, ("conv", 136, 3, 1, 1), ("conv", 72, 3, 1, 1), ("avgpool", 3, 2)), 4, 2),
    "written_out_fc": ({"name": "tiles", "input": (3, 16, 16), "classes": 8,
                        "layers": [("conv", 72, 3, 1, 1), ("conv", 72, 3, 1, 1), ("avgpool", 3, 2), ("fc", 136), ("fc", 8)]}, 40, 1),
}


# the kernels that these take, by layer (asked of the rules, without a GPU): tiles, forms of the strip kernel in the order of its list
REACHES = {
    "wide_96": ("128x128", "96x512"), "wide_88": ("128x128", "96x512"), "wide_256": ("128x128", "256x256"), "wide_200": ("128x128", "256x256"),
    "wide_384": ("strip0", "384x128"), "wide_360": ("strip0", "384x128"),
    "wide_96_splits": ("strip0", "96x512"), "wide_88_splits": ("strip0", "96x512"), "wide_256_splits": ("strip2", "256x256"),
    "wide_200_splits": ("strip2", "256x256"), "wide_384_splits": ("strip2", "384x128"), "wide_360_splits": ("strip2", "384x128"),
    "wide_strided_splits": ("96x512",), "most_splits": ("128x128",), "strided_few_splits": ("128x128",), "strided_one_split": ("gather",),
    "strip_first": ("strip2",), "strip_ragged": ("strip2", "strip2", "strip3"), "strip_small_images": ("strip2", "strip3", "strip0"),
    "strip_two_rows": ("strip2", "strip1"), "strip_no_padding": ("strip2", "strip1"), "strip_groups": ("strip2", "strip1", "strip4"),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_weight_gradient(name):
    nt, mu, lam = CASES[name]
    seed = sum(map(ord, name))
    # every learner's gradient, or the first one's, one's in the middle and the last one's
    learners = range(lam) if mu * lam <= 400 else bounded_learners(nt, lam, mu, seed, 0.1, sorted({0, lam // 2, lam - 1}))
    for (g, rg, loss, rl) in one_gradient(nt, mu, "bf16", seed=seed, scale=0.1, lam=lam, learners=learners):
        check_gradient(nt, "bf16", g, rg, loss, rl, name)
