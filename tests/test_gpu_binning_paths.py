"""The binning's sorting paths against the oracle's lists, bit for bit: one LDS
run, merged runs and counting passes by the planned capacities, digits of
every width by the tile count, at the edges where one path ends and the next
begins; depths drawn from a few values, so most are equal and only a stable
sort keeps the Gaussians' order."""
import numpy as np
import pytest

from gpu_helpers import device_params, log
from oracle.binning import tile_lists
from paper_2512_08498_amd import Rasterizer
from tiny_scenes import camera, scene

pytestmark = pytest.mark.gpu


def _tied_scene(n, depths, seed):
    rng = np.random.default_rng(seed)
    z = rng.choice(np.linspace(2.0, 6.0, depths).astype(np.float32), n)
    means = np.stack([rng.uniform(-0.7, 0.7, n) * z, rng.uniform(-0.6, 0.6, n) * z, z], 1)
    q = rng.standard_normal((n, 4))
    return scene(means, rng.normal(-4.0, 0.5, (n, 3)), q, rng.normal(0.0, 1.5, n), colours=rng.uniform(0, 1, (n, 3)))


RUN, MERGE, BIG = 4096, 16 * 4096, 1 << 23


@pytest.mark.parametrize("n, w, h, ts, cap_rec, cap_pairs", [
    (1, 16, 16, 16, 1, 1),                          # one record, one tile
    (900, 64, 48, 16, RUN, RUN),                    # one run each
    (4096, 64, 48, 32, RUN, RUN + 4096),            # records fill their run, pairs take two
    (4097, 300, 200, 8, RUN + 1, MERGE),            # one item more than a run; 950 tiles in merged runs
    (20000, 300, 200, 16, MERGE, MERGE),            # the last merged capacity
    (20000, 300, 200, 16, MERGE + 1, MERGE + 1),    # the first capacity of the passes; 8-bit tile ids
    (20000, 400, 300, 16, MERGE + 1, 200000),       # 475 tiles: one 9-bit pass
    (20000, 500, 400, 16, MERGE + 1, 200000),       # 800 tiles: one 10-bit pass
    (20000, 700, 500, 16, 90000, 200000),           # 1,408 tiles: one 11-bit pass
    (20000, 730, 720, 16, 90000, 200000),           # 2,070 tiles: two passes
    (20000, 2700, 1600, 8, 90000, 3000000),         # 67,600 tiles: two 9-bit passes
    (20000, 700, 500, 16, BIG - 1, BIG - 1),        # the largest capacity of short chunks
    (20000, 700, 500, 16, BIG, BIG),                # long chunks, an 11-bit pass, searched list bounds
    (20000, 2700, 1600, 8, BIG, BIG),               # the same with 9-bit passes
])
def test_binning_equals_the_oracle(n, w, h, ts, cap_rec, cap_pairs):
    sc, cams = _tied_scene(n, 7, n + w), [camera(0.9 * w, w, h)]
    rast = Rasterizer(cams, n, 0, tile_size=ts, capacity_records=cap_rec, capacity_pairs=cap_pairs)
    params = device_params(sc)
    okeys, ovals, ocsr = tile_lists(sc, cams, ts)
    assert len(okeys) <= cap_pairs
    for _ in range(2):  # the second over what the first left in the workspace
        rast.forward(params)
        rast.check()
        assert rast.capacity == (cap_rec, cap_pairs)  # no re-plan took another path
        keys, vals, csr = rast.debug_binning()
        assert np.array_equal(keys, okeys) and np.array_equal(vals, ovals) and np.array_equal(csr, ocsr)
    log(f"{n} Gaussians, {len(okeys)} pairs, {len(ocsr) - 1} tiles, capacities {cap_rec}/{cap_pairs}: equal")


def test_longest_lists_come_first():
    """The compositing order visits every tile once: an image of many uneven
    tiles equals the same image in tiles of another size."""
    sc, cams = _tied_scene(9000, 50, 3), [camera(700.0, 900, 700), camera(300.0, 333, 211)]
    images = []
    for ts in (8, 16, 32):
        rast = Rasterizer(cams, 9000, 0, tile_size=ts)
        images.append(rast.forward(device_params(sc))["image"].cpu().numpy())
    assert np.array_equal(images[0], images[1]) and np.array_equal(images[0], images[2])
