"""The launch shapes of the server update: vector lengths at both sides of every line between them, with remainders, and window
lengths around the number of gradients a lane keeps in flight, against the same update in fp64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M2 = 1 << 20
CASES = [(1, 1), (3, 5), (4, 16), (255, 17), (257, 2), (600_000, 33), (600_003, 7), (1_500_001, 9), (1_500_005, 4), (6_000_002, 5), (6_000_007, 25),
         (16 * M2 - 1, 32), (16 * M2 + 3, 32), (32 * M2 + 2, 1), (32 * M2 + 6, 5),
         # around the lines of the two-pass form, with stretches that end in part of a block and part of a piece
         (4 * M2 - 1, 45), (4 * M2 + 3, 45), (4 * M2 + 3, 44), (6 * M2 + 4101, 46), (32 * M2, 36), (32 * M2 + 5, 36)]


@pytest.mark.parametrize("P,c", CASES)
@pytest.mark.parametrize("shadow", [False, True])
def test_update_shape(P, c, shadow):
    from paper_1511_05950_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(P % 9973 + c)
    theta = torch.randn(P, device="cuda", generator=gen) * 0.01
    v = torch.randn(P, device="cuda", generator=gen) * 1e-3
    kinds = [torch.randn(P, device="cuda", generator=gen) * 1e-3 for _ in range(min(c, 5))]
    grads = [kinds[l % len(kinds)] for l in range(c)]
    taus = [l % 4 for l in range(c)]
    coef = [float(np.float32(np.float32(0.01) / np.float32(max(t, 1)) / np.float32(c))) for t in taus]
    s = torch.zeros(P, dtype=torch.float64, device="cuda")
    for g, cf in zip(grads, coef):
        s.add_(g.double(), alpha=cf)
    want_v = 0.9 * v.double() + s + sum(coef) * 5e-4 * theta.double()
    want_t = theta.double() - want_v
    for copy_back in (False, True):
        th, vv = theta.clone(), v.clone()
        out = th if copy_back else torch.empty_like(th)
        sh = torch.zeros(P, dtype=torch.bfloat16, device="cuda") if shadow else None
        binding.applyUpdateNoAlloc(th, out, vv, grads, taus, alpha0=0.01, momentum=0.9, weight_decay=5e-4, shadow_out_dev=sh)
        # fp32 chain of c + 2 operations: each rounds by at most 2^-24 of a partial sum, bounded by the sum of magnitudes
        scale = 0.9 * v.abs().double() + sum(cf * g.abs().double() for g, cf in zip(grads, coef)) + theta.abs().double() * 1e-5
        assert bool(((vv.double() - want_v).abs() <= (c + 3) * 2.0 ** -24 * scale + 1e-30).all())
        assert bool(((out.double() - want_t).abs() <= (c + 4) * 2.0 ** -24 * (scale + want_t.abs())).all())
        if shadow:
            assert torch.equal(sh, out.bfloat16())


@pytest.mark.parametrize("P,c", [(1_000_003, 1), (5, 1), (2_000_001, 3)])
def test_fused_passes_take_many_steps(P, c):
    """More deferred updates than one pass takes, at lengths of either kernel variant: the bits of update-by-update launches."""
    from paper_1511_05950_amd import binding
    # a fully connected net of about P parameters whose gradients are written out
    units = max(2, P // 1002)
    net = {"name": "flat", "input": (1, 1, 1000), "classes": 3, "layers": [("fc", units), ("fc", 3)]}
    lam, mu, K = 40 // c * c, 1, 40 // c
    w0 = (np.random.default_rng(1).standard_normal(1004 * units + 3) * 0.01).astype(np.float32)
    gen = torch.Generator(device="cuda").manual_seed(P)
    x = torch.randn((lam, 1, 1, 1000), device="cuda", generator=gen)
    y = torch.randint(0, 3, (lam,), device="cuda", dtype=torch.int32, generator=gen)
    out = []
    for flags in (0, binding.FLAG_EAGER_UPDATES):
        ctx = binding.Sasgd(lam, mu, lam // c, 1, net=net, compute="fp32", alpha0=0.01, momentum=0.9, weight_decay=1e-3,
                            init_weights=w0, flags=flags)
        for l in range(lam):
            ctx.getMinibatch(l, x[l:l + 1], y[l:l + 1])
            ctx.pullWeights(l)
        ctx.calcGradient(list(range(lam)))
        ctx.setProfiling(True)
        for l in range(lam):
            ctx.pushGradient(l)
            if (l + 1) % c == 0:
                ctx.sumGradients()
                ctx.applyUpdate()
        _, passes = ctx.phaseTime(2)
        assert passes == (K if flags else (K + 31) // 32)
        out.append((ctx.copyWeights(), ctx.copyMomentum()))
        ctx.destroy()
    for a, b in zip(*out):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
