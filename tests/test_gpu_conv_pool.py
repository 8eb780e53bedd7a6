"""A first convolution and the 3 x 3 / 2 max pooling behind it, which share a kernel in bf16, against the CPU oracle and, bit by bit, against the
same layers in separate kernels: 8 channels and multiples of 16, one to four blocks of 32 output channels and ones that end inside,
rows in even and odd numbers, windows that the image cuts, rounds that are not full, images in one piece and in several, ReLU in front and behind."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_net import SPREAD_FACTOR, TOL, draw_case, layer_errors, one_gradient

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

R, P, F = ("relu",), ("maxpool", 3, 2), ("fc", 16)


def net(c, h, w, *layers):
    return {"name": "conv_pool", "input": (c, h, w), "classes": 16, "layers": list(layers) + [F]}


CASES = {
    # name: (network, mini-batch size, learners)
    "c8_32": (net(3, 32, 32, ("conv", 32, 5, 1, 2), P, R), 8, 32),
    "c8_32_relu": (net(3, 31, 33, ("conv", 32, 5, 1, 2), R, P), 8, 32),
    "c8_40": (net(5, 20, 64, ("conv", 40, 3, 1, 0), R, P), 8, 32),
    "c8_24_few_images": (net(3, 66, 46, ("conv", 24, 3, 1, 1), P), 2, 24),
    "c16_64": (net(12, 28, 27, ("conv", 64, 3, 1, 1), R, P), 6, 32),
    "c16_128": (net(9, 17, 30, ("conv", 128, 3, 1, 1), P, R), 6, 32),
    "strided_96": (net(3, 59, 63, ("conv", 96, 11, 4, 0), R, P), 8, 32),
    "strided_72": (net(3, 43, 83, ("conv", 72, 7, 2, 0), P, R), 4, 32),
    "long_rows": (net(3, 9, 120, ("conv", 16, 3, 1, 1), R, P), 6, 32),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_against_oracle(name):
    nt, mu, lam = CASES[name]
    for (g, rg, loss, rl, eg) in one_gradient(nt, mu, "bf16", seed=sum(map(ord, name)), scale=0.05, lam=lam, both=True, learners=[0, lam - 1]):
        # a winner that rounding decides moves a term of its tensor's sums: as far as the oracle's own two evaluations lie apart
        _, spread = layer_errors(nt, rg, eg)
        _, errs = layer_errors(nt, g, rg)
        assert all(e < max(TOL["bf16"], SPREAD_FACTOR * sp) for e, sp in zip(errs, spread)), (name, errs, spread)
        assert abs(loss - rl) < 1e-3 * max(1.0, abs(rl))


@pytest.mark.parametrize("relu_first", [True, False])
@pytest.mark.parametrize("odd_values", [False, True], ids=["plain", "inf_nan_zero"])
def test_same_bits_as_separate_kernels(relu_first, odd_values):
    """Images of eight channels of bf16 values behind a 1 x 1 convolution that copies them: the pooled one is the second layer there, in kernels
    of its own, and everything behind it has the same bits.  NaNs (infinite pixels become some in the copy) and images of zeros pass as they do there."""
    from paper_1511_05950_amd import binding
    tail = [("conv", 40, 3, 1, 1)] + ([R, P] if relu_first else [P, R])
    one, two = net(8, 25, 30, *tail), net(8, 25, 30, ("conv", 8, 1, 1, 0), *tail)
    lam, mu = 16, 16
    w, X, Y = draw_case(one, lam, mu, 9, 0.05)
    X = torch.from_numpy(X).cuda().bfloat16().float()
    if odd_values:
        r = torch.rand(X.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
        X[r < 2e-4], X[(r > 2e-4) & (r < 3e-4)], X[(r > 3e-4) & (r < 4e-4)] = float("nan"), float("inf"), float("-inf")
        X[:mu] = 0
        # a copying convolution would spread a NaN or an infinity over its pixel's other channels: the pixel is that value in all of them
        bad = X.sum(1, keepdim=True)
        X = torch.where(torch.isfinite(bad), X, bad.expand_as(X) * torch.ones_like(X))
    Yd = torch.from_numpy(Y).cuda()
    copy = np.concatenate([np.eye(8, dtype=np.float32).ravel(), np.zeros(8, np.float32), w])
    got = []
    for nt, theta in ((one, w), (two, copy)):
        ctx = binding.Sasgd(lam, mu, lam, 2, net=nt, compute="bf16", init_weights=theta)
        loss, rank = torch.zeros(lam, device="cuda"), None
        for k in range(lam):
            ctx.getMinibatch(k, X[k * mu:(k + 1) * mu], Yd[k * mu:(k + 1) * mu])
            ctx.pullWeights(k, 0)
        ctx.calcGradient(list(range(lam)), loss)
        tail_size = wl.num_params(one) - 40 * 8 * 9 - 40          # the layers behind the pooling
        got.append((loss.cpu(), [ctx.copyGradient(k)[-tail_size:] for k in range(lam)]))
        ctx.destroy()
    if not odd_values:
        assert torch.equal(got[0][0], got[1][0])
    else:
        np.testing.assert_array_equal(got[0][0].numpy(), got[1][0].numpy())
    for a, b in zip(got[0][1], got[1][1]):
        np.testing.assert_array_equal(a, b)                       # NaNs in the same places count as equal


@pytest.mark.parametrize("tail", [(P,), (R, P), (P, R)], ids=["pool", "relu_pool", "pool_relu"])
def test_infinities_reach_the_pooling(tail):
    """As above, with pixels of 3e38 in one channel, which the copying convolution keeps as they are: the pooled one, whose filters weigh that channel
    with 2 (even ones) or -2 everywhere, makes infinities of both signs.  Behind the pooling a 1 x 1 convolution with weights below zero (even channels)
    or above and a ReLU make zeros of those of positive pixels, and the learner's loss is finite; of negative pixels' it is not.  Other learners
    have NaN pixels, which that ReLU ends."""
    from paper_1511_05950_amd import binding
    behind = list(tail) + [("conv", 16, 1, 1, 0), R]
    one, two = net(8, 25, 30, ("conv", 40, 3, 1, 1), *behind), net(8, 25, 30, ("conv", 8, 1, 1, 0), ("conv", 40, 3, 1, 1), *behind)
    lam, mu = 16, 16
    w, X, Y = draw_case(one, lam, mu, 9, 0.05)
    first = w[:40 * 8 * 9].reshape(40, 8, 9)
    first[0::2, 0], first[1::2, 0] = 2, -2
    second = w[40 * 8 * 9 + 40:][:16 * 40].reshape(16, 40)
    second[:, 0::2], second[:, 1::2] = -np.abs(second[:, 0::2]), np.abs(second[:, 1::2])
    X = torch.from_numpy(X).bfloat16().float().view(lam, mu, 8, 25, 30)
    g = torch.Generator().manual_seed(3)
    spots = torch.rand((lam, mu, 25, 30), generator=g) < 2e-2
    X[1::4, :, 0][spots[1::4]], X[2::4, :, 0][spots[2::4]] = 3e38, -3e38
    X[3::4] = X[3::4].masked_fill(spots[3::4][:, :, None], float("nan"))
    for k, reach in enumerate([(False, False, False), (True, True, False), (True, True, False), (False, False, True)]):   # what the pooling reads
        y = torch.nn.functional.conv2d(X[k], torch.from_numpy(first).view(40, 8, 3, 3), torch.from_numpy(w[40 * 8 * 9:][:40]), padding=1)
        assert (bool((y == np.inf).any()), bool((y == -np.inf).any()), bool(y.isnan().any())) == reach
    X, Yd = X.view(lam * mu, 8, 25, 30).cuda(), torch.from_numpy(Y).cuda()
    copy = np.concatenate([np.eye(8, dtype=np.float32).ravel(), np.zeros(8, np.float32), w])
    got = []
    for nt, theta in ((one, w), (two, copy)):
        ctx = binding.Sasgd(lam, mu, lam, 2, net=nt, compute="bf16", init_weights=theta)
        loss = torch.zeros(lam, device="cuda")
        for k in range(lam):
            ctx.getMinibatch(k, X[k * mu:(k + 1) * mu], Yd[k * mu:(k + 1) * mu])
            ctx.pullWeights(k, 0)
        ctx.calcGradient(list(range(lam)), loss)
        got.append((loss.cpu().numpy(), [ctx.copyGradient(k)[40 * 8 * 9 + 40 - wl.num_params(one):] for k in range(lam)]))
        ctx.destroy()
    assert np.isfinite(got[0][0]).tolist() == [k % 4 != 2 for k in range(lam)]
    np.testing.assert_array_equal(got[0][0], got[1][0])
    for a, b in zip(got[0][1], got[1][1]):
        np.testing.assert_array_equal(a, b)
