"""A record whose tiles the plan does not have stops the forward with the
internal code 3 before anything is written for it, on plans of every size."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from gpu_helpers import log
from paper_2512_08498_amd import _lib

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(_lib.LIB_PATH), "csrc")


@pytest.fixture(scope="module")
def binning(tmp_path_factory):
    import torch
    torch.zeros(1, device="cuda")  # the HIP runtime that the library is to share
    _lib.load()
    so = str(tmp_path_factory.mktemp("driver") / "binning_driver.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I/opt/rocm/include", "-I" + CSRC, "-I" + os.path.join(HERE, "..", "include"), "-o", so,
                    os.path.join(HERE, "binning_driver.cpp"), _lib.LIB_PATH], check=True)
    lib = C.CDLL(so)

    def run(t_tot, cap_pairs, rects):
        r = np.array(rects, np.uint32)
        out = np.zeros(1 + t_tot, np.uint32)
        assert lib.run_binning(t_tot, 64, cap_pairs, len(r), C.c_void_p(r.ctypes.data), C.c_void_p(out.ctypes.data)) == 0
        return int(out[0]), out[1:]

    return run


def _rect(tile, w=1, h=1, pitch=8):
    return ((w - 1) << 16, (h - 1) << 16, tile, pitch)


# one LDS run, merged runs, counting passes, and list bounds by search
@pytest.mark.parametrize("cap_pairs", [4096, 65536, 65537, 1 << 23])
def test_tiles_outside_the_plan(binning, cap_pairs):
    good = [_rect(0), _rect(63), _rect(5, 3, 2), _rect(0, 8, 8)]
    code, lens = binning(64, cap_pairs, good)
    want = np.ones(64, np.uint32)
    want[[0, 63, 5, 6, 7, 13, 14, 15]] += 1
    assert code == 0 and np.array_equal(lens, want)
    # past the last tile by one (whose low bits are tile 0's), by a row, by far,
    # and past the end of 32 bits
    for bad in (_rect(64), _rect(63, 2, 1), _rect(56, 8, 2), _rect(1000), _rect(0xFFFFFFFF), _rect(0xFFFFFFFF, 2, 1)):
        code, _ = binning(64, cap_pairs, good[:2] + [bad] + good[2:])
        log(f"capacity {cap_pairs}: first tile {bad[2]}, code {code}")
        assert code == 3, bad
