"""calcGradient of small networks and mini-batches at the edges of the kernels' tiles, against the CPU oracle: positions and
channels beside multiples of 16, 32 and 128, channel counts that are no multiple of four, every window size, pooling of both
kinds in front of another convolution and of the fully connected layers, contractions of the fully connected layers split over
workgroups, and numbers of learners around the lines between the tile shapes."""
import pytest

import workloads as wl
from oracle import cnn
from test_gpu_net import check_gradient, decided_seed, draw_case, one_gradient

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def net(c, h, w, classes, *layers):
    return {"name": "small", "input": (c, h, w), "classes": classes, "layers": list(layers) + [("fc", classes)]}


R = ("relu",)
NETS = {
    # name: (network, mini-batch size, learners)
    "one_position": (net(1, 1, 1, 2, ("conv", 1, 1, 1, 0)), 1, 1),
    "windows_2_4": (net(2, 9, 11, 3, ("conv", 5, 2, 1, 0), R, ("avgpool", 2, 2), ("conv", 7, 4, 1, 2), ("maxpool", 3, 2), R), 3, 2),
    "windows_7_3": (net(5, 23, 18, 7, ("conv", 17, 7, 2, 3), R, ("maxpool", 3, 2), ("conv", 31, 3, 1, 1), R, ("avgpool", 3, 2)), 2, 3),
    "window_11": (net(3, 31, 35, 4, ("conv", 33, 11, 4, 0), R, ("conv", 13, 3, 1, 1), ("avgpool", 3, 2), R, ("fc", 19), R), 2, 2),
    "hidden_split": (net(3, 22, 22, 5, ("conv", 21, 3, 1, 1), R, ("maxpool", 3, 2), ("fc", 37), R, ("fc", 18), R), 17, 2),
    "no_pooling": (net(4, 6, 7, 6, ("conv", 9, 3, 1, 1), R, ("conv", 12, 3, 1, 1), R), 5, 2),
    # pooling windows other than 3 x 3 / 2, four channels at a time and one, clipped at the border, and of stride 1
    "max_4_3": (net(3, 20, 17, 5, ("conv", 12, 3, 1, 1), R, ("maxpool", 4, 3), ("conv", 9, 3, 1, 1), R, ("maxpool", 4, 2)), 3, 2),
    "max_2_2": (net(3, 15, 18, 5, ("conv", 9, 3, 1, 1), R, ("maxpool", 2, 2), ("conv", 12, 3, 1, 1), R, ("maxpool", 5, 3)), 3, 2),
    "stride_1": (net(3, 10, 9, 5, ("conv", 12, 3, 1, 1), R, ("maxpool", 2, 1), ("conv", 9, 3, 1, 1), R, ("avgpool", 2, 1)), 2, 2),
    "max_1_1": (net(3, 9, 9, 5, ("conv", 8, 3, 1, 1), ("maxpool", 1, 2), R, ("conv", 5, 3, 1, 1), R, ("maxpool", 2, 1)), 2, 2),
    # hidden layers whose products are split over workgroups: both directions, rows of 16 bytes, one image and more than 16;
    # the input gradient alone with weights that start between 16-byte pieces
    "fc_split_1": (net(2, 12, 12, 6, ("conv", 16, 3, 1, 1), R, ("fc", 2052), R), 1, 1),
    "fc_split_17": (net(2, 12, 12, 6, ("conv", 16, 3, 1, 1), R, ("fc", 2052), R), 17, 1),
    "fc_split_unaligned": (net(2, 8, 12, 6, ("conv", 6, 3, 1, 1), R, ("maxpool", 2, 2), ("fc", 2052), R), 17, 1),
    "large_tiles": (net(3, 17, 16, 5, ("conv", 36, 5, 1, 2), R, ("maxpool", 3, 2), ("conv", 34, 3, 1, 1), R), 15, 16),
    # flattened inputs of many pixels per channel (no ReLU: every sum is decided): index times pixels is beyond 2^32
    "flat_160x160": (net(3, 160, 160, 10, ("conv", 8, 3, 1, 1), ("fc", 64)), 2, 1),
    "flat_112x112": (net(2, 112, 112, 5, ("conv", 64, 3, 1, 1), ("fc", 4)), 2, 2),
    "wide_tiles": (net(3, 26, 24, 5, ("conv", 33, 3, 1, 1), R, ("conv", 30, 3, 1, 1), R, ("avgpool", 3, 2)), 32, 2),
}


@pytest.mark.parametrize("compute", ["fp32", "bf16"])
@pytest.mark.parametrize("name", sorted(NETS))
def test_gradient(name, compute):
    nt, mu, lam = NETS[name]
    seed = sum(map(ord, name))
    scale = 0.02 if name.startswith("flat") else 0.3     # sums of 10^5 terms: scores stay around one
    if compute == "fp32":
        seed = decided_seed(nt, lam, mu, seed, scale)
    for (g, rg, loss, rl) in one_gradient(nt, mu, compute, seed=seed, lam=lam, scale=scale):
        check_gradient(nt, compute, g, rg, loss, rl, name)


@pytest.mark.parametrize("compute", ["fp32", "bf16"])
def test_ranks(compute):
    from paper_1511_05950_amd import binding
    nt, mu, lam = NETS["windows_7_3"]
    theta, X, Y = draw_case(nt, lam, mu, 11, 0.3)
    ctx = binding.Sasgd(lam, mu, lam, 2, net=nt, compute=compute, init_weights=theta)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    loss, rank = torch.zeros(lam, device="cuda"), torch.zeros(lam * mu, dtype=torch.int32, device="cuda")
    for k in range(lam):
        ctx.getMinibatch(k, Xd[k * mu:(k + 1) * mu], Yd[k * mu:(k + 1) * mu])
        ctx.pullWeights(k)
    ctx.evaluate(list(range(lam)), loss, rank)
    _, scores = cnn.class_scores(nt, theta, X, Y, round_bf16=compute == "bf16")
    spread = 1e-4 if compute == "fp32" else 2e-2
    for i, z in enumerate(scores):
        # a score within rounding of the label's may fall on either side of it
        near = abs(z - z[Y[i]]) <= spread * abs(z).max()
        lo = int(((z > z[Y[i]]) & ~near).sum())
        assert lo <= int(rank[i]) <= lo + int(near.sum()) - 1
    ctx.destroy()
