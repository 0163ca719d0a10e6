"""X of an image is the same bits whatever it is planned with, so that a
render and its ground truth compare equal when their pixels are."""
import numpy as np
import pytest
import torch

from gpu_helpers import log
from paper_2512_08498_amd import Frequency

pytestmark = pytest.mark.gpu

SIZES = [(640, 360)] * 16 + [(960, 540)] * 4 + [(1, 1), (45, 27), (7, 2560), (2560, 5), (800, 525), (320, 180),
                                                (1600, 900), (100, 1), (64, 48), (1280, 720), (375, 81), (480, 270)]


def _images(rng, sizes):
    return [torch.from_numpy(rng.uniform(0, 1, 3 * w * h).astype(np.float32)).cuda() for w, h in sizes]


def test_an_image_alone_and_in_batches():
    rng = np.random.default_rng(17)
    imgs = _images(rng, SIZES)
    alone = torch.cat([Frequency([s]).significance(i) for s, i in zip(SIZES, imgs)])
    for extra in ([], [(1600, 900)] * 6, [(64, 48)] * 300):
        X = Frequency(SIZES + extra).significance(torch.cat(imgs + _images(rng, extra)))[:len(SIZES)]
        differ = [SIZES[i] for i in torch.nonzero(alone != X).flatten().tolist()]
        log(f"{len(SIZES)} images and {len(extra)} others: {len(differ)} differ {differ}")
        assert not differ
