"""The compositing walks that a launch's size chooses between give the same
results: the forward's groups of two and four records bit for bit, on lists
that end at every remainder of a group and a 64-entry step, with pixels that
stop in them and tiles cut by the image's edge."""
import numpy as np
import pytest
import torch

from gpu_helpers import device_params, log
from paper_2512_08498_amd import Rasterizer
from tiny_scenes import camera, scene

pytestmark = pytest.mark.gpu


def _stack(n, seed, opacity_mean, w, h, f):
    """n Gaussians in front of one camera, denser towards the image's left, so
    its tiles' lists have many different lengths."""
    rng = np.random.default_rng(seed)
    z = rng.uniform(2.0, 6.0, n)
    x = (rng.beta(1.0, 3.0, n) - 0.5) * w / f
    means = np.stack([x * z, rng.uniform(-0.5, 0.5, n) * h / f * z, z], 1)
    q = rng.standard_normal((n, 4))
    return scene(means, rng.normal(-3.4, 0.6, (n, 3)), q, rng.normal(opacity_mean, 2.0, n),
                 colours=rng.uniform(0, 1, (n, 3)))


@pytest.mark.parametrize("ts", [8, 16, 32])
@pytest.mark.parametrize("n, opacity_mean", [(0, 0.0), (1, 2.0), (65, 1.0), (3000, 3.0)])
def test_forward_groups_agree_bitwise(ts, n, opacity_mean):
    w, h, f = 133, 101, 120.0
    one = camera(f, w, h)
    sc = _stack(n, 5 + n, opacity_mean, w, h, f)
    params = device_params(sc)
    few = Rasterizer([one], n, 0, tile_size=ts, bg=(0.2, 0.4, 0.6))
    a = few.forward(params)
    # the same view in a batch of more than 40,960 waves: the others look away
    away = [camera(f, 1664, 1664, R=np.diag([1.0, -1.0, -1.0])) for _ in range(2)]
    many = Rasterizer([one] + away, n, 0, tile_size=ts, bg=(0.2, 0.4, 0.6), capacity_records=max(n, 1),
                      capacity_pairs=max(200 * n, 1))
    b = many.forward(params)
    px = w * h
    for k, size in (("image", 3 * px), ("t_final", px), ("last_pos", px), ("n_contrib", px)):
        assert torch.equal(a[k][:size], b[k][:size]), k
    if n == 3000:
        assert int((a["t_final"] < 2e-4).sum()) > 50  # pixels that stopped
    log(f"ts {ts}, {n} Gaussians: longest walk {int(a['last_pos'].max())}, {int(a['n_contrib'].max())} composited")
