"""The dense Adam step at the edges of its workgroups (groups of 0 to a few
values past a multiple of 1,024, whose later groups are not 16-byte aligned)
and on both sides of the size from which it bypasses the caches, against the
same formula in double precision.  The second bias correction, 1 - 0.999^t, is
a float32 difference near 1e-3: its rounding of 2^-24 is up to 1e-4 of a step
of at most the learning rate, and the parameter takes one rounding per step."""
import pytest
import torch

from paper_2512_08498_amd import FusedAdam, Rasterizer
from tiny_scenes import camera

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, degree", [(1, 0), (3, 1), (341, 0), (342, 3), (1023, 2), (1024, 0), (1025, 3),
                                       (474_575, 3), (474_577, 3)])
def test_adam_sizes(n, degree):
    k, steps = (degree + 1) ** 2, 2
    lr = (1e-2, 2e-2, 3e-2, 4e-2, 5e-2, 6e-2)
    shapes = dict(mean=(3, n), log_scale=(3, n), quat=(4, n), opacity_logit=(n,), sh=(k, 3, n))
    g = torch.Generator("cuda").manual_seed(n)
    params = {a: torch.randn(s, generator=g, device="cuda") for a, s in shapes.items()}
    grads = {a: torch.randn(s, generator=g, device="cuda") for a, s in shapes.items()}
    before = {a: t.double() for a, t in params.items()}
    opt = FusedAdam(Rasterizer([camera()], n, degree), params, lr=lr)
    for _ in range(steps):
        opt.apply(grads)
    b1, b2, eps = 0.9, 0.999, 1e-15
    for i, a in enumerate(shapes):
        p, d = before[a], grads[a].double()
        rate = torch.full_like(p, lr[i])
        if a == "sh":
            rate[1:] = lr[5]
        m, v = torch.zeros_like(p), torch.zeros_like(p)
        for t in range(1, steps + 1):
            m, v = b1 * m + (1 - b1) * d, b2 * v + (1 - b2) * d * d
            p = p - rate * (m / (1 - b1**t)) / ((v / (1 - b2**t)).sqrt() + eps)
        bound = steps * (1e-4 * float(rate.max()) + float(p.abs().max()) * 2.0**-24)
        assert float((params[a].double() - p).abs().max()) <= bound, a


@pytest.mark.parametrize("n, degree", [(271_186, 3), (271_187, 3), (813_560, 3), (1_142_858, 0)])
def test_fused_step_past_the_caches(n, degree):
    """The fused step at the sizes from which its moments, then its parameters
    pass the caches by, against the backward and the dense step (the same
    formula on the same gradients), and the next forward, which reads what the
    step has written."""
    g = torch.Generator("cuda").manual_seed(n)
    k = (degree + 1) ** 2

    def normal(*shape, sd=1.0):
        return torch.randn(*shape, generator=g, device="cuda") * sd

    params = dict(mean=normal(3, n), log_scale=normal(3, n, sd=0.3) - 5.0, quat=normal(4, n), opacity_logit=normal(n),
                  sh=normal(k, 3, n, sd=0.3))
    params["mean"][2] += 5.0
    rast = Rasterizer([camera(f=200.0, w=160, h=120)], n, degree, capacity_pairs=20 * n)
    out = rast.forward(params)
    dl = normal(3 * rast.total_px, sd=1e-4)
    grads = rast.backward(params, out, dl)
    apart = {a: t.clone() for a, t in params.items()}
    dense = FusedAdam(rast, apart)
    dense.apply(grads)
    fused = FusedAdam(rast, params)
    rast.backward_adam(params, out, dl, fused)
    for a in params:
        assert torch.allclose(params[a], apart[a], rtol=0, atol=1e-7), a
        assert torch.equal(fused.m[a], dense.m[a]), a
    assert torch.allclose(rast.forward(params)["image"], rast.forward(apart)["image"], rtol=0, atol=1e-4)
