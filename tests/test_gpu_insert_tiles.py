"""LoG insertion at the edges of its tiles and of its compaction: views whose
sides end at, before and after a 64 x 32 tile (whole interior tiles, rows that
are not 16-byte aligned, sides below a filter's width), more views than a
wave's lanes, and more pixels than the blocks whose counts the writing kernel
adds itself.  Tolerances as for the other sizes; the compaction is exact."""
import numpy as np
import pytest
import torch

from paper_2512_08498_amd import Rasterizer
from test_gpu_insert import _cams, _check

pytestmark = pytest.mark.gpu


def _inputs(sizes, seed):
    rng = np.random.default_rng(seed)
    gts = [rng.uniform(0, 1, (3, h, w)).astype(np.float32) for w, h in sizes]
    rds = [(g * rng.uniform(0, 1)).astype(np.float32) for g in gts]
    depths = [rng.uniform(1, 5, (h, w)).astype(np.float32) for w, h in sizes]
    return gts, rds, depths


@pytest.mark.parametrize("sigma", [0.3, 0.6, 1.0, 1.3, 5.0 / 3.0])
@pytest.mark.parametrize("sizes", [[(192, 32), (256, 65), (200, 33), (201, 64), (64, 31), (5, 70), (3, 2), (196, 96)],
                                   [(12 + v % 5, 9 + v % 3) for v in range(70)]])
def test_insert_at_the_tiles_edges(sizes, sigma):
    _check(_cams(sizes, 31), *_inputs(sizes, 32), sigma=sigma, tau=0.1)


@pytest.mark.parametrize("sizes", [[(64, 64)], [(1023, 4096), (1, 4096)], [(1024, 4096)] * 4, [(1024, 4096)] * 4 + [(7, 1)]])
def test_insert_compaction(sizes):
    rast = Rasterizer(_cams(sizes, 33), 1, 0)
    n = sum(w * h for w, h in sizes)
    g = torch.Generator("cuda").manual_seed(34)
    gt, rd = (torch.rand(3 * n, generator=g, device="cuda") for _ in range(2))
    res = rast.log_insert(gt, rd, torch.rand(n, generator=g, device="cuda") + 1.0, sigma=0.6, tau_a=0.4, p_render=True)
    want = torch.nonzero((res["p_gt"] - res["p_render"]).clamp_min(0) > np.float32(0.4).item()).flatten()
    assert int(res["count"]) == len(want) > 0
    assert torch.equal(res["pix"][: len(want)].long(), want)
