"""A colour that is not finite reaches the pixels that composite its record,
and the gradients of what those pixels composite in front of it, and nothing
else, in every walk that a launch's size or its tuning chooses."""
import numpy as np
import pytest
import torch

from gpu_helpers import device_params, log
from paper_2512_08498_amd import Rasterizer
from tiny_scenes import camera, scene

pytestmark = pytest.mark.gpu

NEVER = 0xFFFFFFFF
W, H, F, N = 133, 101, 120.0, 1500


def _scene(spoiled=None):
    """Opaque enough for pixels to stop; `spoiled` Gaussians' red is infinite."""
    rng = np.random.default_rng(31)
    z = rng.uniform(2.0, 6.0, N)
    means = np.stack([rng.uniform(-0.6, 0.6, N) * W / F * z, rng.uniform(-0.6, 0.6, N) * H / F * z, z], 1)
    sc = scene(means, rng.normal(-2.9, 0.6, (N, 3)), rng.standard_normal((N, 4)), rng.normal(1.0, 2.0, N),
               colours=rng.uniform(0, 1, (N, 3)))
    params = device_params(sc)
    if spoiled is not None:
        params["sh"].view(-1, N)[0, torch.from_numpy(spoiled).cuda()] = float("inf")
    return sc, params


def _spoiled():
    return np.sort(np.random.default_rng(8).choice(N, 40, replace=False))


def _reached(ts, spoiled):
    """The pixels that composite a spoiled record: those it colours when it
    alone has a colour."""
    sc, params = _scene()
    sh = params["sh"].view(-1, N)
    sh[:] = -0.5 / 0.28209479177387814
    sh[:, torch.from_numpy(spoiled).cuda()] = 1.0
    r = Rasterizer([camera(F, W, H)], N, 0, tile_size=ts)
    return (r.forward(params)["image"][:W * H] > 1e-6).cpu().numpy()


@pytest.mark.parametrize("ts", [8, 16, 32])
def test_images(ts):
    spoiled = _spoiled()
    _, params = _scene(spoiled)
    one = camera(F, W, H)
    few = Rasterizer([one], N, 0, tile_size=ts).forward(params)
    away = [camera(F, 1664, 1664, R=np.diag([1.0, -1.0, -1.0])) for _ in range(2)]
    many = Rasterizer([one] + away, N, 0, tile_size=ts, capacity_records=N, capacity_pairs=400 * N).forward(params)
    a, b = few["image"][:3 * W * H].cpu().numpy(), many["image"][:3 * W * H].cpu().numpy()
    reached = _reached(ts, spoiled)
    log(f"ts {ts}: {int(reached.sum())} pixels composite a spoiled record, {int((~np.isfinite(a)).sum())} and "
        f"{int((~np.isfinite(b)).sum())} values are not finite")
    assert 100 < reached.sum() < W * H - 100
    assert np.array_equal(np.isfinite(b[:W * H]), ~reached)
    assert np.array_equal(a, b, equal_nan=True)
    assert np.isfinite(a[W * H:]).all()  # green and blue


def test_gradients():
    """Against the one-wave walk, which switches lanes off that do not
    composite a record."""
    spoiled = _spoiled()
    _, params = _scene(spoiled)
    dl = torch.from_numpy(np.random.default_rng(5).uniform(0.1, 1.0, 3 * W * H).astype(np.float32)).cuda()

    def grads(ts, long_list):
        r = Rasterizer([camera(F, W, H)], N, 0, tile_size=ts, long_list=long_list)
        g = r.backward(params, r.forward(params), dl)
        return {k: v.double().cpu().numpy() for k, v in g.items() if v is not None}

    ref = grads(16, NEVER)
    spoiled_g = ~np.isfinite(ref["opacity_logit"].reshape(-1))
    log(f"{int(spoiled_g.sum())} Gaussians in front of a spoiled one")
    assert len(spoiled) <= spoiled_g.sum() < N // 2
    for ts, long_list in ((16, 1024), (16, 0), (16, 20), (8, 1024), (32, 1024)):
        got = grads(ts, long_list)
        for k, a in ref.items():
            fin = np.isfinite(a)
            assert np.array_equal(fin, np.isfinite(got[k])), (ts, long_list, k, int((~fin).sum()),
                                                              int((~np.isfinite(got[k])).sum()))
            # the order of the sums and the colours' origin differ, as without spoiled colours
            d = np.linalg.norm(got[k][fin] - a[fin]) / np.linalg.norm(a[fin])
            assert d <= 1e-5, (ts, long_list, k, d)
