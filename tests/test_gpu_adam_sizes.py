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
