"""The library's host code on fake HIP calls (fake_hip.cpp, in a process of its
own; no GPU): the launch grids of the persistent schedule, and readers of the
counters on streams of their own."""
import ctypes as C
import importlib.util
import os
import subprocess
import sys
import threading

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2512_08498_amd", "libgsr.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libgsr.so not built (run __graft_entry__.build())")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.cpp"),
                    "-ldl", "-lpthread"], check=True)
    return so


def _run(fake, case):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), fake, case], capture_output=True, text=True,
                       timeout=100, cwd=ROOT)
    assert r.returncode == 0, r.stdout + r.stderr


def test_persistent_grids_fit_their_kernels(fake):
    """A persistent launch has the workgroups that its own kernel keeps on the
    device, whichever kernels were launched before, on each device."""
    _run(fake, "grids")


def test_a_second_reader_of_the_counters_keeps_to_its_stream(fake):
    """gsr_check in two threads on two streams, the first one's not done: the
    second returns at once, with the counters of its own workspace, and copies
    on its own stream only (the null stream waits for the first one's where
    that blocks, and later work on it for this copy)."""
    _run(fake, "readers")


# ---- in the process with the fake calls

def _load(fake):
    f = C.CDLL(fake, mode=C.RTLD_GLOBAL)
    f.fake_text.restype = C.c_char_p
    f.fake_hold.argtypes = [C.c_void_p]
    path = os.path.join(ROOT, "paper_2512_08498_amd", "_lib.py")  # by itself: the package imports torch
    spec = importlib.util.spec_from_file_location("gsr_lib", path)
    L = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(L)
    return f, L, L.load()


def _plan(L, lib, ts, w, h, persistent=1, n=8):
    ctx = C.c_void_p()
    assert lib.gsr_create(C.byref(ctx)) == 0
    assert lib.gsr_set_tuning(ctx, C.byref(L.Tuning(ts, 1024, persistent, 0.0))) == 0
    cams = (L.Camera * 1)()
    cams[0].R[0] = cams[0].R[4] = cams[0].R[8] = 1.0
    cams[0].fx = cams[0].fy = 100.0
    cams[0].cx, cams[0].cy = w / 2, h / 2
    cams[0].width, cams[0].height = w, h
    size, pix = C.c_size_t(), (C.c_int64 * 2)()
    opts = L.PlanOptions(ts, n, n, (C.c_float * 3)())
    assert lib.gsr_plan(ctx, cams, 1, n, 0, C.byref(opts), C.byref(size), pix) == 0, lib.gsr_last_error(ctx)
    raw = (C.c_char * (size.value + 256))()
    ws = (C.addressof(raw) + 255) // 256 * 256
    return ctx, cams, ws, size.value, raw


def _grids(fake):
    f, L, lib = _load(fake)
    mem = (C.c_float * 4096)()
    p = C.cast(mem, C.c_void_p)
    seen = {}
    for device in (0, 1):
        f.fake_device(device)
        for ts, w, h in ((16, 64, 48), (16, 1664, 1664), (8, 64, 48), (8, 2048, 2048), (32, 64, 48), (32, 4096, 4096)):
            ctx, cams, ws, size, raw = _plan(L, lib, ts, w, h)
            g = L.Gaussians(8, 0, *[C.cast(p, f) for _, f in L.Gaussians._fields_[2:]])
            out = L.FwdOut(*[C.cast(p, f) for _, f in L.FwdOut._fields_])
            grads = L.Grads(*[C.cast(p, f) for _, f in L.Grads._fields_])
            f.fake_clear()
            args = (ctx, C.byref(g), p, 1, C.c_void_p(ws), size)
            assert lib.gsr_render_forward(*args, C.byref(out), None) == 0, lib.gsr_last_error(ctx)
            assert lib.gsr_render_backward(*args, C.byref(out), p, C.byref(grads), 0, None) == 0
            launches = [line.split() for line in f.fake_text().decode().splitlines() if "k_raster_" in line]
            assert len(launches) == 2, launches
            for _, name, grid, block, resident in launches:
                print(device, ts, w, name, grid, block, resident)
                assert int(grid) == (16 + 8 * device) * int(resident) // 8 * 8, (ts, w, name, grid, resident)
                seen[name] = block
    assert len(seen) == 6 + 4, seen  # the forwards' two groups, the backwards of 16 px few and many


def _readers(fake):
    f, L, lib = _load(fake)
    ctx, cams, ws, size, raw = _plan(L, lib, 16, 64, 48)
    second = (C.c_char * (size + 256))()
    ws2 = (C.addressof(second) + 255) // 256 * 256
    (C.c_uint32 * 3).from_address(ws)[:] = [3, 5, 0]
    (C.c_uint32 * 3).from_address(ws2)[:] = [7, 9, 0]

    def read(w, stream, into):
        c = [C.c_int64() for _ in range(3)]
        assert lib.gsr_required_capacity(ctx, C.c_void_p(w), *[C.byref(x) for x in c], C.c_void_p(stream)) == 0
        into[:] = [c[0].value, c[1].value]

    a, b, alone = [], [], []
    read(ws, 16, alone)
    f.fake_hold(32)
    t = threading.Thread(target=read, args=(ws, 32, a))
    t.start()
    assert f.fake_wait_until_held()
    f.fake_clear()
    read(ws2, 48, b)
    copies = f.fake_text().decode().splitlines()
    assert not a, "the first reader's stream was not done"
    f.fake_release()
    t.join()
    print(alone, a, b, copies)
    assert (alone, a, b) == ([3, 5], [3, 5], [7, 9])
    assert copies == ["copy on stream 48"]


if __name__ == "__main__":
    {"grids": _grids, "readers": _readers}[sys.argv[2]](sys.argv[1])
