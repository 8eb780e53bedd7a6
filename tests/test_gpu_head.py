"""The last fully connected layer, loss and input gradient in one kernel behind the layer-by-layer kernels, against the CPU oracle: behind an average pooling
(with and without a ReLU), a max pooling, a convolution and a hidden layer, with few and with many images in a call (fewer lanes each)."""
import pytest

import workloads as wl
from test_gpu_net import check_gradient, decided_seed, one_gradient

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

A = ("avgpool", 3, 2)


def net(*layers, classes=10):
    return {"name": "head", "input": (3, 13, 12), "classes": classes, "layers": [("conv", 64, 5, 1, 2)] + list(layers) + [("fc", classes)]}


NETS = {"avgpool": net(A), "two_pools": net(A, A, classes=3), "convolution": net(A, ("conv", 16, 3, 1, 1), classes=7),
        "hidden": net(A, ("fc", 64), classes=50)}


@pytest.mark.parametrize("lam, mu", [(64, 6), (64, 20)])
@pytest.mark.parametrize("compute", ["fp32", "bf16"])
@pytest.mark.parametrize("name", sorted(NETS))
def test_gradient(name, compute, lam, mu):
    nt = NETS[name]
    seed = 3 * mu + len(name)
    for (g, rg, loss, rl) in one_gradient(nt, mu, compute, seed=seed, scale=0.1, lam=lam, learners=[0, 31, 63]):
        check_gradient(nt, compute, g, rg, loss, rl, name)


def test_relu_behind_the_pooling():
    nt = net(A, ("relu",))
    seed = decided_seed(nt, 64, 6, 30, 0.1)      # no ReLU input so near zero that its sign depends on the order of a sum
    for (g, rg, loss, rl) in one_gradient(nt, 6, "fp32", seed=seed, scale=0.1, lam=64, learners=[0, 31, 63]):
        check_gradient(nt, "fp32", g, rg, loss, rl, "relu")


@pytest.mark.parametrize("compute", ["fp32", "bf16"])
def test_evaluation_has_the_losses_of_the_gradient_pass(compute):
    from paper_1511_05950_amd import binding, driver
    nt, lam, mu = NETS["avgpool"], 40, 30
    w0 = wl.init_weights(nt, 3, std=0.1)
    X, Y = torch.from_numpy(wl.images(nt, lam * mu, 4)).cuda(), torch.from_numpy(wl.labels(nt, lam * mu, 5)).cuda()
    ctx = binding.Sasgd(lam, mu, lam, 2, net=nt, compute=compute, init_weights=w0)
    loss, got, rank = torch.zeros(lam, device="cuda"), torch.zeros(lam, device="cuda"), torch.full((lam * mu,), -1, dtype=torch.int32, device="cuda")
    for k in range(lam):
        ctx.getMinibatch(k, X[k * mu:(k + 1) * mu], Y[k * mu:(k + 1) * mu])
        ctx.pullWeights(k, 0)
    ctx.calcGradient(list(range(lam)), loss)
    driver.evaluate(ctx, X, Y, lam, mu, got, rank)
    assert torch.equal(loss, got)
    assert int(rank.min()) >= 0 and int(rank.max()) < 10 and 3 < float(rank.float().mean()) < 6      # near-random weights
    ctx.destroy()
