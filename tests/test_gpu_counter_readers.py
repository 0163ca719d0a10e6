"""Several threads read the counters of workspaces of one plan at once, each on
a stream of its own: every reading is its workspace's."""
import ctypes as C
import threading

import pytest
import torch

from gpu_helpers import device_params, log
from paper_2512_08498_amd import Rasterizer
from tiny_scenes import mini_rig

pytestmark = pytest.mark.gpu


def test_concurrent_readers():
    sc, cams = mini_rig()
    rast = Rasterizer(cams, sc.n, sc.sh_degree)
    rast.forward(device_params(sc))
    torch.cuda.synchronize()
    base = [C.c_int64() for _ in range(3)]
    read = rast.lib.gsr_required_capacity
    assert read(rast.ctx, C.c_void_p(rast.workspace.data_ptr()), *[C.byref(x) for x in base], rast.stream()) == 0
    # copies of the workspace, with other counts
    copies = [rast.workspace.clone() for _ in range(4)]
    for i, w in enumerate(copies):
        w[:8].view(torch.int32).add_(i)
    torch.cuda.synchronize()
    wrong = []

    def reader(i, stream):
        c = [C.c_int64() for _ in range(3)]
        for _ in range(300):
            st = read(rast.ctx, C.c_void_p(copies[i].data_ptr()), *[C.byref(x) for x in c], C.c_void_p(stream))
            got = (st, c[0].value, c[1].value)
            if got != (0, base[0].value + i, base[1].value + i):
                wrong.append((i, got))

    streams = [torch.cuda.Stream() for _ in copies]
    threads = [threading.Thread(target=reader, args=(i, s.cuda_stream)) for i, s in enumerate(streams)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    log(f"{base[0].value} records, {base[1].value} pairs; {len(wrong)} wrong readings")
    assert base[0].value > 0 and not wrong, wrong[:5]
