"""Re-layout of a mini-batch's images, bf16: long rows of a space-to-depth first layer, in pieces; the row kernel against the kernel
with a lane per pixel, which takes over where images lie at an address that is no multiple of 16, to the bit; with a pixel mean and
without; images of a few pixels, several in a workgroup."""
import numpy as np
import pytest

from test_gpu_net import check_gradient, draw_case, one_gradient

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def net(h, w, *layers):
    return {"name": "layout", "input": (3, h, w), "classes": 8, "layers": list(layers) + [("avgpool", 3, 2), ("fc", 24), ("fc", 8)]}


STRIDED = ("conv", 16, 11, 4, 0)
# widths of 640, 641 and 1 281 pixels after space-to-depth: one, two and three pieces; images cut in the last row of pixels
WIDE = {"one_piece": net(19, 2560, STRIDED), "two_pieces": net(22, 2564, STRIDED), "three_pieces": net(21, 5124, STRIDED)}


def gradients(nt, mu, theta, X, Y, shift, mean):
    from paper_1511_05950_amd import binding
    buf = torch.zeros(X.size + 4, device="cuda")
    x = buf[shift:shift + X.size].view(X.shape)
    x.copy_(torch.from_numpy(X))
    y = torch.from_numpy(Y).cuda()
    lam = X.shape[0] // mu
    ctx = binding.Sasgd(lam, mu, lam, 2, net=nt, compute="bf16", init_weights=theta)
    if mean is not None:
        ctx.setPixelMean(torch.from_numpy(mean).cuda())
    for k in range(lam):
        ctx.getMinibatch(k, x[k * mu:(k + 1) * mu], y[k * mu:(k + 1) * mu])
        ctx.pullWeights(k)
    ctx.calcGradient(range(lam))
    out = [ctx.copyGradient(k) for k in range(lam)]
    ctx.destroy()
    return out


@pytest.mark.parametrize("name", sorted(WIDE))
def test_long_rows(name):
    nt, mu, lam = WIDE[name], 2, 24
    for (g, rg, loss, rl) in one_gradient(nt, mu, "bf16", seed=sum(map(ord, name)), scale=0.1, lam=lam)[::23]:
        check_gradient(nt, "bf16", g, rg, loss, rl, name)


@pytest.mark.parametrize("nt, mu, lam", [(WIDE["two_pieces"], 2, 24), (net(47, 44, STRIDED), 16, 24)], ids=["two_pieces", "one_piece"])
def test_rows_and_pixels_have_the_same_bits(nt, mu, lam):
    theta, X, Y = draw_case(nt, lam, mu, 7, 0.1)
    mean = np.random.default_rng(8).standard_normal(nt["input"]).astype(np.float32)
    for m in (None, mean):
        for a, b in zip(gradients(nt, mu, theta, X, Y, 0, m), gradients(nt, mu, theta, X, Y, 1, m)):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32)) and np.abs(a).max() > 0
    # the mean is subtracted before anything is rounded
    assert np.array_equal(gradients(nt, mu, theta, X - mean, Y, 0, None)[0], gradients(nt, mu, theta, X, Y, 0, mean)[0])


@pytest.mark.parametrize("h, w, mu, lam", [(5, 3, 70, 6), (3, 3, 300, 2), (4, 9, 64, 8)])
def test_images_of_a_few_pixels(h, w, mu, lam):
    nt = net(h, w, ("conv", 72, 3, 1, 1))
    for (g, rg, loss, rl) in one_gradient(nt, mu, "bf16", seed=h * w, scale=0.1, lam=lam):
        check_gradient(nt, "bf16", g, rg, loss, rl, (h, w))
