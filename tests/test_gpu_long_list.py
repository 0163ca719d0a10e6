"""gsr_tuning.long_list is the list length it says, in batches of any size: the
16 px tiles with at least that many entries take the four-wave walk of the
backward, the others the one-wave walk, and 1024 leaves the choice to the
library.  The walks add a record's terms in another order, so a Gaussian whose
tiles are all on one side of the length has the bits of that walk alone.  The
lengths are those at which a step of the longest-first order begins (16 steps
per octave), as the long lists are a prefix of it."""
import numpy as np
import pytest
import torch

from gpu_helpers import device_params, log
from paper_2512_08498_amd import Rasterizer
from tiny_scenes import camera, scene

pytestmark = pytest.mark.gpu

NEVER, LIBRARY = 0xFFFFFFFF, 1024


def _case(w, h, n, seed):
    rng = np.random.default_rng(seed)
    f = 0.9 * w
    z = rng.uniform(2.0, 6.0, n)
    x = (rng.beta(1.0, 3.0, n) - 0.5) * w / f  # denser towards the left
    means = np.stack([x * z, rng.uniform(-0.5, 0.5, n) * h / f * z, z], 1)
    q = rng.standard_normal((n, 4))
    sc = scene(means, rng.normal(-3.4 - np.log(w / 133), 0.6, (n, 3)), q, rng.normal(1.0, 2.0, n),
               colours=rng.uniform(0, 1, (n, 3)))
    return sc, camera(f, w, h)


def _step(length):
    """The least length of its step of the order."""
    unit = 1 << max(length.bit_length() - 5, 0)
    return max(length // unit * unit, 2)


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("w, h, n", [(133, 101, 3000),        # 63 tiles
                                     (1693, 1301, 120_000)])  # 8,692 tiles
def test_the_length_is_the_one_that_was_set(w, h, n, persistent):
    sc, cam = _case(w, h, n, w)
    params = device_params(sc)
    dl = torch.from_numpy(np.random.default_rng(3).uniform(-1, 1, 3 * w * h).astype(np.float32)).cuda()
    lists = {}

    def grads(long_list):
        r = Rasterizer([cam], n, 0, tile_size=16, long_list=long_list, persistent=persistent,
                       capacity_records=n, capacity_pairs=200 * n)
        assert r.tuning()["long_list"] == long_list
        g = r.backward(params, r.forward(params), dl)
        torch.cuda.synchronize()
        if not lists:
            lists["keys"], lists["vals"], lists["csr"] = r.debug_binning()
        return np.concatenate([v.reshape(-1, n).cpu().numpy() for v in g.values() if v is not None])

    one, four = grads(NEVER), grads(2)
    csr, vals = lists["csr"].astype(np.int64), lists["vals"]
    lens = np.diff(csr)
    shortest = np.full(n, 1 << 40)  # per Gaussian, over its tiles
    longest = np.zeros(n, np.int64)
    np.minimum.at(shortest, vals, np.repeat(lens, lens))
    np.maximum.at(longest, vals, np.repeat(lens, lens))
    apart = (one != four).any(0)
    live = np.sort(lens[lens > 0])
    lengths = [_step(int(live[len(live) // 4])), _step(int(live[len(live) // 2])), _step(int(live[9 * len(live) // 10])), _step(int(live[-1])),
               int(live[-1]) + 1]
    cases = [(length, length) for length in lengths]
    if len(lens) > 6144:  # the library's rule: at least 32 entries and a 4096th of all pairs
        assert len(vals) // 4096 in range(32, 128, 4)
        cases += [(0, 0), (LIBRARY, len(vals) // 4096)]
    else:  # the library's rule: every list
        assert np.array_equal(grads(LIBRARY), grads(0))
    for value, length in cases:
        got = grads(value)
        above, below = shortest >= max(length, 2), (longest < length) & (longest > 0)
        assert np.array_equal(got[:, above], four[:, above]), (value, length)
        assert np.array_equal(got[:, below], one[:, below]), (value, length)
        log(f"{w}x{h} long_list {value}: {int((above & apart).sum())} Gaussians of long lists and "
            f"{int((below & apart).sum())} of short ones, whose walks differ")
        if length == lengths[1]:
            assert (above & apart).any() and (below & apart).any()
