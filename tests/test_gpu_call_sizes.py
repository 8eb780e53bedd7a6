"""Networks with layers that have no matrix-instruction kernel of their own, at both sides of the line between the two executors of a
call: large calls layer by layer (hidden layers' gradients as factors in bf16), small ones on the compact kernels (every gradient
written out), in one context.  No ReLU and no max-pooling: nothing that rounding decides."""
import numpy as np
import pytest

import workloads as wl
from oracle import cnn, protocol
from test_gpu_net import check_gradient, draw_case, one_gradient, rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

A = ("avgpool", 3, 2)
ODD_HIDDEN = {"name": "odd_hidden", "input": (3, 16, 16), "classes": 10,
              "layers": [("conv", 64, 3, 1, 1), A, ("conv", 64, 3, 1, 1), A, ("fc", 64), ("fc", 37), ("fc", 10)]}
ODD_CONV = {"name": "odd_conv", "input": (3, 20, 20), "classes": 10,
            "layers": [("conv", 30, 5, 1, 2), A, ("conv", 50, 3, 1, 1), A, ("fc", 64), ("fc", 10)]}


class Run:
    def __init__(self, net, compute, lam, mu, n, seed, flags=0):
        from paper_1511_05950_amd import binding
        self.net, self.compute, self.lam, self.mu = net, compute, lam, mu
        self.theta, self.X, self.Y = draw_case(net, lam, mu, seed, 0.1)
        self.Xd, self.Yd = torch.from_numpy(self.X).cuda(), torch.from_numpy(self.Y).cuda()
        self.ctx = binding.Sasgd(lam, mu, n, 4, net=net, compute=compute, alpha0=0.01, momentum=0.9, weight_decay=1e-3, init_weights=self.theta,
                                 flags=flags)
        self.loss = torch.zeros(lam, device="cuda")

    def calc(self, learners):
        for k in learners:
            self.ctx.getMinibatch(k, self.Xd[k * self.mu:(k + 1) * self.mu], self.Yd[k * self.mu:(k + 1) * self.mu])
            self.ctx.pullWeights(k)
        self.ctx.calcGradient(learners, self.loss)

    def check(self, learner, place, tag):
        s = slice(learner * self.mu, (learner + 1) * self.mu)
        loss, g = cnn.loss_and_gradient(self.net, self.theta, self.X[s], self.Y[s], round_bf16=self.compute == "bf16")
        got = self.ctx.copyGradient(learner)
        check_gradient(self.net, self.compute, got, g, float(self.loss[place]), loss, tag)
        return got


@pytest.mark.parametrize("net, compute, lam, mu", [(ODD_HIDDEN, "bf16", 8, 32), (ODD_HIDDEN, "bf16", 5, 70), (ODD_HIDDEN, "fp32", 16, 48),
                                                   (ODD_CONV, "bf16", 16, 32), (ODD_CONV, "fp32", 16, 32)],
                         ids=["odd_hidden-bf16", "odd_hidden-bf16-written_out", "odd_hidden-fp32", "odd_conv-bf16", "odd_conv-fp32"])
def test_large_and_small_calls(net, compute, lam, mu):
    r = Run(net, compute, lam, mu, lam, seed=5)
    # the hidden layer's gradient of a large call stays factors (mini-batches of up to 32 images, bf16)
    assert (r.ctx.factoredParams() > 0) == (net is ODD_HIDDEN and compute == "bf16" and mu <= 32)
    r.calc(list(range(lam)))
    for k in (0, lam - 1):
        r.check(k, k, "large call")
    r.calc([1])
    r.check(1, 0, "small call")
    r.calc(list(range(lam)))
    r.check(1, 1, "large call again")
    r.ctx.destroy()


def test_window_of_both_kinds():
    """One update of a gradient held as factors and a written-out one, the next of factors alone, applied in one pass; then an
    update of written-out gradients alone."""
    r = Run(ODD_HIDDEN, "bf16", 8, 32, 4, seed=9)
    r.calc(list(range(8)))
    grads = {k: r.ctx.copyGradient(k) for k in (0, 2, 3)}
    r.calc([1])
    grads[1] = r.ctx.copyGradient(1)
    th, v = r.theta.astype(np.float64), np.zeros(r.theta.size)
    for window, taus in (((0, 1), (0, 0)), ((2, 3), (1, 1))):
        for k, tau in zip(window, taus):
            assert r.ctx.pushGradient(k) == tau
        r.ctx.sumGradients()
        r.ctx.applyUpdate()
        th, v = protocol.server_update(th, v, [grads[k] for k in window], taus, 0.01, 0.9, 1e-3)
    assert rel(r.ctx.copyWeights() - r.theta, th - r.theta) < 1e-4 and rel(r.ctx.copyMomentum(), v) < 1e-5
    r.calc([4])
    r.calc([5])
    late = [r.ctx.copyGradient(k) for k in (4, 5)]
    for k in (4, 5):
        r.ctx.pushGradient(k)
    r.ctx.sumGradients()
    r.ctx.applyUpdate()
    th, v = protocol.server_update(th, v, late, (0, 0), 0.01, 0.9, 1e-3)
    assert rel(r.ctx.copyWeights() - r.theta, th - r.theta) < 1e-4 and rel(r.ctx.copyMomentum(), v) < 1e-5
    r.ctx.destroy()


def test_one_pass_over_both_kinds_has_the_bits_of_separate_launches():
    """Windows of factors, of both kinds and of written-out gradients (which take another kernel when they are alone)."""
    from paper_1511_05950_amd import binding
    out = []
    for flags in (0, binding.FLAG_EAGER_UPDATES):
        r = Run(ODD_HIDDEN, "bf16", 8, 32, 4, seed=9, flags=flags)
        r.calc(list(range(8)))
        for k in (1, 4, 5):
            r.calc([k])
        for window in ((0, 1), (2, 3), (4, 5), (6, 7)):
            for k in window:
                r.ctx.pushGradient(k)
            r.ctx.sumGradients()
            r.ctx.applyUpdate()
        out.append((r.ctx.copyWeights(), r.ctx.copyMomentum(), r.ctx.copyWeights(2)))
        r.ctx.destroy()
    for a, b in zip(*out):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


DEEP = {"name": "deep", "input": (8, 3, 3), "classes": 10, "layers": [("conv", 512, 3, 1, 1)] * 9 + [("fc", 10)]}


def test_partial_gradients_are_bounded():
    """Split weight gradients of nine 512-channel convolutions: 20 M parameters, so 32 partial copies of each would take 2.4 GB a
    learner.  With fewer copies (two images and fewer splits than tiles) the gradients are the oracle's."""
    from paper_1511_05950_amd import binding
    lib = binding.load()
    sizes, held = [], {}

    def alloc(size, _):
        sizes.append(size)
        t = torch.empty(size, dtype=torch.uint8, device="cuda")
        held[t.data_ptr()] = t
        return t.data_ptr()

    def release(address, _):
        del held[address]

    hooks = binding.ALLOC_FN(alloc), binding.RELEASE_FN(release)
    cfg = binding.SasgdConfig()
    cfg.lambda_, cfg.mu, cfg.n, cfg.ring_depth, cfg.net, cfg.num_layers = 1, 32, 1, 1, binding.NET_CUSTOM, 10
    layers = (binding.SasgdLayer * 10)(*[(0, 512, 3, 1, 1)] * 9, (4, 10, 0, 0, 0))
    cfg.layers, cfg.in_channels, cfg.in_height, cfg.in_width = layers, 8, 3, 3
    cfg.alloc, cfg.release = hooks
    w0 = torch.zeros(wl.num_params(DEEP), device="cuda")
    h = binding.ctypes.c_void_p()
    assert lib.sasgd_create(binding.ctypes.byref(cfg), w0.data_ptr(), binding.ctypes.byref(h)) == binding.OK
    lib.sasgd_destroy(h)
    assert not held and max(sizes) < 160 << 20          # the workspace: 128 MiB of partial sums and a few MiB of activations

    for (g, rg, loss, rl) in one_gradient(DEEP, 2, "fp32", seed=3, scale=0.015, lam=1):
        check_gradient(DEEP, "fp32", g, rg, loss, rl, "deep")
