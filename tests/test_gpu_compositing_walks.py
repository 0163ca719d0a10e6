"""The compositing walks that a launch's size chooses between give the same
results: the forward's groups of two and four records bit for bit, on lists
that end at every remainder of a group and a 64-entry step, with pixels that
stop in them and tiles cut by the image's edge; the backward's walks up to the
order of their sums."""
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


def _grads(sc, params, cam, ts, long_list, spoil, persistent=False):
    rast = Rasterizer([cam], sc.n, sc.sh_degree, tile_size=ts, long_list=long_list, persistent=persistent,
                      capacity_records=max(sc.n, 1), capacity_pairs=max(200 * sc.n, 1))
    out = rast.forward(params)
    rng = np.random.default_rng(9)
    dl = rng.uniform(-1.0, 1.0, (3, cam.height, cam.width)).astype(np.float32)
    if spoil:  # one pixel's gradient is not finite
        dl[:, cam.height // 2, cam.width // 4] = (np.nan, np.inf, -np.inf)
    g = rast.backward(params, out, torch.from_numpy(dl.reshape(-1)).cuda())
    return {k: v.double().cpu().numpy() for k, v in g.items() if v is not None}


@pytest.mark.parametrize("w, h, n, spoil", [(133, 101, 0, False), (133, 101, 1, False), (133, 101, 65, False),
                                            (133, 101, 3000, False), (133, 101, 3000, True),
                                            (1693, 1301, 160_000, False), (1693, 1301, 160_000, True)])
def test_backward_walks_agree(w, h, n, spoil):
    """A wave per 16 px tile (at 1693 x 1301, of more than 6,144 tiles, nearly
    all lists, as none holds a 4096th of the pairs; with long_list 5 those
    under 5 entries) and a wave per 8 x 8 block (long_list 0, the smaller
    image, and the other tile sizes) form the same terms per pixel and add them
    in another order: up to 24 additions of 2^-24 each, 1.4e-6 of the absolute
    terms, seven times that for their cancellation.  A pixel whose gradient is
    not finite reaches the Gaussians it composited and no others, in every
    walk."""
    f = 120.0 * w / 133
    cam = camera(f, w, h)
    sc = _stack(n, 11 + n, 2.0, w, h, f)
    if n > 3000:
        sc.log_scale[:] -= 1.2
    params = device_params(sc)
    ref = _grads(sc, params, cam, 16, 1024, spoil)
    queued = _grads(sc, params, cam, 16, 1024, spoil, persistent=True)
    assert all(np.array_equal(ref[k], queued[k], equal_nan=True) for k in ref)
    for ts, long_list in ((16, 0), (16, 5), (8, 1024), (32, 1024)):
        got = _grads(sc, params, cam, ts, long_list, spoil)
        for k, a in ref.items():
            fin = np.isfinite(a)
            assert np.array_equal(fin, np.isfinite(got[k])), (ts, long_list, k)
            if n > 1:
                assert fin.all() != spoil, k
            d = np.linalg.norm(got[k][fin] - a[fin]) / max(np.linalg.norm(a[fin]), 1e-30)
            assert d <= 1e-5, (ts, long_list, k, d)
    log(f"{w}x{h}, {n} Gaussians, spoil {spoil}: " + ", ".join(f"{k} {int(np.isfinite(v).sum())}" for k, v in ref.items()))
