"""One-pass updates from the factors of fully connected gradients (bf16): written-out products and updates against runs whose gradients are
written out by the weight-gradient kernels, which test_gpu_net.py compares with the oracle.  Many gradients of up to 16 images (operands
straight from memory, half a k-block and a whole one), mini-batches that pass through LDS in one to four stages with remainders
of 8 to 56 images, layers that end inside a tile, few and many tiles."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_net import rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NET = {"name": "factors", "input": (3, 12, 12), "classes": 8,                       # 1 152 -> 4 104 -> 264 -> 8: large enough for the layer-by-layer
      # kernels, which keep factors, at every size below
       "layers": [("conv", 32, 3, 1, 1), ("avgpool", 3, 2), ("fc", 4104), ("relu",), ("fc", 264), ("relu",), ("fc", 8)]}


def one_update(lam, mu, flags, net=NET):
    from paper_1511_05950_amd import binding
    w0 = wl.init_weights(net, 5, std=0.05)
    X, Y = torch.from_numpy(wl.images(net, lam * mu, 6)).cuda(), torch.from_numpy(wl.labels(net, lam * mu, 7)).cuda()
    ctx = binding.Sasgd(lam, mu, 1, 2, net=net, compute="bf16", alpha0=0.05, momentum=0.5, weight_decay=1e-2, init_weights=w0, flags=flags)
    assert (ctx.factoredParams() > 0) == (flags == 0)
    for update in range(2):
        for k in range(lam):
            ctx.getMinibatch(k, X[k * mu:(k + 1) * mu], Y[k * mu:(k + 1) * mu])
            ctx.pullWeights(k, 0)
        ctx.calcGradient(list(range(lam)))
        if update == 0:
            grads = [ctx.copyGradient(k) for k in sorted({0, lam - 1})]
        for k in range(lam):
            ctx.pushGradient(k)
        ctx.sumGradients()
        ctx.applyUpdate()
        if update == 0:
            w, v = ctx.copyWeights(), ctx.copyMomentum()
    out = grads, w, v, ctx.copyWeights(), w0
    ctx.destroy()
    return out


@pytest.mark.parametrize("lam, mu", [(8, 8), (12, 16), (20, 13), (64, 4), (12, 20), (5, 32), (1, 100), (1, 136), (1, 200), (1, 256), (3, 190), (4, 256)])
def test_update_from_factors(lam, mu):
    from paper_1511_05950_amd import binding
    fa, fl = one_update(lam, mu, 0), one_update(lam, mu, binding.FLAG_FLAT_FC_GRADIENT)
    # the same operands and 32-bit sums in another order: n products of magnitude a sum to within n eps a of each other at most, and to
    # within a few eps of the norm on average
    for a, b in zip(fa[0], fl[0]):
        assert rel(a, b) < 1e-5
    w0 = fa[4].astype(np.float64)
    assert rel(fa[1] - w0, fl[1] - w0) < 1e-5
    assert rel(fa[2], fl[2]) < 1e-5
    # element by element, over every tensor's own size
    pos = 0
    for shape, nb in wl.param_shapes(NET):
        for n in (int(np.prod(shape)), nb):
            a, b = fa[2][pos:pos + n].astype(np.float64), fl[2][pos:pos + n].astype(np.float64)
            assert np.max(np.abs(a - b)) <= 1e-4 * np.max(np.abs(b)), (shape, n)
            pos += n
    assert rel(fa[3] - w0, fl[3] - w0) < 2e-3          # a second update, on weights that differ in the last place


class Buffer:
    """A learner's gradient buffer, whose address was asked for at some time, as a tensor."""

    def __init__(self, ctx, learner):
        self.__cuda_array_interface__ = {"data": (ctx.gradientPtr(learner), False), "shape": (ctx.P,), "typestr": "<f4", "version": 2}


@pytest.mark.parametrize("asked", ["at_the_start", "after_calcGradient", "after_pushGradient"])
def test_a_caller_that_holds_the_gradient_finds_and_changes_it_there(asked):
    """Mini-batches of more than 32 images: a buffer whose address the caller has holds every later gradient without another call, and the
    update takes what the caller made of it, as where all gradients are written out."""
    from paper_1511_05950_amd import binding
    lam, mu = 2, 40
    w0 = wl.init_weights(NET, 15, std=0.05)
    X, Y = torch.from_numpy(wl.images(NET, lam * mu, 16)).cuda(), torch.from_numpy(wl.labels(NET, lam * mu, 17)).cuda()
    got = []
    for flags in (0, binding.FLAG_FLAT_FC_GRADIENT):
        ctx = binding.Sasgd(lam, mu, 1, 2, net=NET, compute="bf16", alpha0=0.05, momentum=0.5, weight_decay=1e-2, init_weights=w0, flags=flags)
        assert (ctx.factoredParams() > 0) == (flags == 0)
        held, seen = None, []
        if asked == "at_the_start":
            held = torch.as_tensor(Buffer(ctx, 0), device="cuda")
        for update in range(2):
            for k in range(lam):
                ctx.getMinibatch(k, X[k * mu:(k + 1) * mu], Y[k * mu:(k + 1) * mu])
                ctx.pullWeights(k, 0)
            ctx.calcGradient(list(range(lam)))
            if held is None and asked == "after_calcGradient":
                held = torch.as_tensor(Buffer(ctx, 0), device="cuda")
            for k in range(lam):
                ctx.pushGradient(k)
            if held is None:
                held = torch.as_tensor(Buffer(ctx, 0), device="cuda")
            seen.append(held.clone())
            held.clamp_(-1e-4, 1e-4)                          # the caller's clipping
            seen.append(held.clone())
            ctx.sumGradients()
            ctx.applyUpdate()
            seen.append(torch.from_numpy(ctx.copyMomentum()))
        got.append([s.cpu().numpy() for s in seen])
        del held
        ctx.destroy()
    assert np.abs(got[0][0]).max() > 2e-4                     # there was something to clip
    for k, (a, b) in enumerate(zip(*got)):
        # (sums in another order where the factors had been taken; behind the first update, weights that differ in the last place)
        assert rel(a, b) < (1e-5 if k < 3 else 2e-3), (asked, k)


WIDER = {"name": "factors", "input": (3, 12, 12), "classes": 8,           # 1 152 -> 12 296 -> 264: layer by layer for one learner of 33 images too
         "layers": [("conv", 32, 3, 1, 1), ("avgpool", 3, 2), ("fc", 12296), ("relu",), ("fc", 264), ("relu",), ("fc", 8)]}


@pytest.mark.parametrize("mu", [33, 40, 64])
def test_update_from_factors_of_one_learner(mu):
    """Three and four k-blocks, which a lone gradient takes through the tiles of 32 x 32 weights; bounds as above."""
    from paper_1511_05950_amd import binding
    fa, fl = one_update(1, mu, 0, WIDER), one_update(1, mu, binding.FLAG_FLAT_FC_GRADIENT, WIDER)
    w0 = fa[4].astype(np.float64)
    assert rel(fa[0][0], fl[0][0]) < 1e-5 and rel(fa[1] - w0, fl[1] - w0) < 1e-5 and rel(fa[2], fl[2]) < 1e-5


@pytest.mark.parametrize("mu", [40, 64, 176, 177, 256])
@pytest.mark.parametrize("n_factored", [1, 3])
def test_factors_of_many_images_beside_a_written_out_gradient(mu, n_factored):
    """A window of learners' gradients and one pushed from outside in the middle of them, at both sides of the line beyond which the factors are written
    out first; a second window finds the learners' buffers as the first one left them."""
    from paper_1511_05950_amd import binding
    lam = n_factored + 1
    w0 = wl.init_weights(NET, 25, std=0.05)
    X, Y = torch.from_numpy(wl.images(NET, lam * mu, 26)).cuda(), torch.from_numpy(wl.labels(NET, lam * mu, 27)).cuda()
    outside = (torch.randn(wl.num_params(NET), generator=torch.Generator().manual_seed(28)) * 1e-3).cuda()
    ctx = binding.Sasgd(lam, mu, 1, 2, net=NET, compute="bf16", alpha0=0.05, momentum=0.5, weight_decay=1e-2, init_weights=w0)
    assert ctx.factoredParams() > 0
    theta, v = w0.astype(np.float64), 0.0
    for window in range(2):
        ks = list(range(n_factored))
        for k in ks:
            ctx.getMinibatch(k, X[(k + window) * mu:(k + window + 1) * mu], Y[(k + window) * mu:(k + window + 1) * mu])
            ctx.pullWeights(k, 0)
        ctx.calcGradient(ks)
        for k in ks[:1]:
            ctx.pushGradient(k)
        ctx.pushGradientExternal(outside, ctx.timestamp())
        for k in ks[1:]:
            ctx.pushGradient(k)
        ctx.sumGradients()
        ctx.applyUpdate()
        got, got_v = ctx.copyWeights(), ctx.copyMomentum()
        g = sum(ctx.copyGradient(k).astype(np.float64) for k in ks) + outside.cpu().numpy()     # (what the update read, written out)
        v = 0.5 * v + 0.05 / lam * g + 0.05 * 1e-2 * theta
        theta = theta - v
        assert rel(got_v, v) < 1e-5 and rel(got, theta) < 1e-7, window          # (32-bit weights, each rounded once)
        theta, v = got.astype(np.float64), got_v.astype(np.float64)
    ctx.destroy()
