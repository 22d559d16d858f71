"""Which requests of an admission share a launch (on the CPU, with stand-in
cameras), and that frames of several height classes in one launch equal the
oracle bit for bit (GPU)."""

import types

import numpy as np
import pytest

from paper_1610_04124_amd import serving


def executor(classes, num_cu=256, max_frames=8, layout=None):
    """An executor's grouping state without a device: cameras (width, height, D)."""
    ex = object.__new__(serving.GpuExecutor)
    ex.cameras = [types.SimpleNamespace(handle=types.SimpleNamespace(D=d), ncols=lambda w=w: w // 5,
                                        height_class=lambda h=h: (h + 63) // 64, height=h)
                  for w, h, d in classes]
    ex.max_frames, ex.num_cu, ex.layout, ex.classes = max_frames, num_cu, layout or {}, {}
    for c in ex.cameras:
        k = c.height_class()
        hm, dm, cm = ex.classes.get(k, (0, 0, 0))
        ex.classes[k] = (max(hm, c.height), max(dm, c.handle.D), max(cm, c.ncols()))
    return ex


def groups(ex, cams):
    return [(k, [r.camera for r in m])
            for k, m in ex.grouped([serving.Request(i, c, None, 0.0) for i, c in enumerate(cams)])]


TALL, MID, LOW = 12, 7, 4
CAMERAS = [(1024, 440, 128), (1280, 720, 128), (640, 240, 128)]


def test_short_admissions_share_a_launch():
    assert groups(executor(CAMERAS), [0, 1, 0]) == [(TALL, [1, 0, 0])]
    assert groups(executor(CAMERAS), [2, 0, 1]) == [(TALL, [1, 0, 2])]
    assert groups(executor(CAMERAS), [0, 2]) == [(MID, [0, 2])]
    assert groups(executor(CAMERAS), [0, 0]) == [(MID, [0, 0])]


@pytest.mark.parametrize("num_cu,want", [(74, [(TALL, [1, 0, 0])]), (73, [(TALL, [1]), (MID, [0, 0])])])
def test_columns_per_compute_unit(num_cu, want):
    # 256 + 2 * 204 = 664 columns: 9 of each of 74 compute units hold them
    assert groups(executor(CAMERAS, num_cu=num_cu), [0, 1, 0]) == want


@pytest.mark.parametrize("num_cu,want", [(56, [(MID, [0, 2])]), (55, [(MID, [0]), (LOW, [2])])])
def test_columns_per_compute_unit_below_513_rows(num_cu, want):
    # 204 + 128 = 332 columns: 6 of each of 56 compute units hold them
    assert groups(executor(CAMERAS, num_cu=num_cu), [0, 2]) == want


def test_limits_of_the_taller_class():
    # the taller class's batch holds max_frames frames of its own column count
    narrow = [(1024, 440, 128), (300, 720, 128)]
    assert groups(executor(narrow), [1, 0, 0]) == [(TALL, [1, 0, 0])]
    assert groups(executor(narrow), [1, 0, 0, 0]) == [(TALL, [1]), (MID, [0, 0, 0])]
    # its frames and its disparities
    assert groups(executor(CAMERAS, max_frames=2), [0, 1, 0]) == [(TALL, [1]), (MID, [0, 0])]
    deep = [(1024, 440, 256), (1280, 720, 128)]
    assert groups(executor(deep), [0, 1]) == [(TALL, [1]), (MID, [0])]
    # a tuned layout keeps its class apart
    assert groups(executor(CAMERAS, layout={MID: (1, 2, 0)}), [0, 1]) == [(TALL, [1]), (MID, [0])]


def test_costs_off_the_grid_keep_classes_apart():
    # one frame off the grid would take the whole launch off the spread kernel
    for off in ([0], [1], [0, 1]):
        ex = executor(CAMERAS)
        for c in off:
            ex.cameras[c].handle.on_grid = False
        assert groups(ex, [0, 1]) == [(TALL, [1]), (MID, [0])]
        # the classes below it may still join each other
        want = [(TALL, [1]), (MID, [0]), (LOW, [2])] if 0 in off else [(TALL, [1]), (MID, [0, 2])]
        assert groups(ex, [0, 1, 2]) == want


@pytest.mark.gpu
def test_handles_say_whether_costs_are_on_the_grid():
    import synth
    import paper_1610_04124_amd as P
    for g in (-1, 0, 10):
        h = P.Stixels(synth.make_params(max_width=64, max_height=32, flags=1, cost_grid_log2=g))
        assert h.on_grid == (g >= 0)
        h.close()


@pytest.mark.gpu
def test_mixed_heights_in_one_launch_equal_oracle():
    import torch
    import oracle
    import synth
    import paper_1610_04124_amd as P
    from gpu_helpers import announce, assert_frames_equal, to_device

    cams, params = [], []
    for w, h, d in [(200, 150, 64), (330, 530, 128), (97, 64, 32)]:
        p = synth.make_params(camera=synth.camera_for_size(w, h), stixel_width=5,
                              max_disparity=d, max_width=w, max_height=h, flags=1)
        params.append(p)
        cams.append(serving.CameraSpec(P.Stixels(p), w, h))
    ex = serving.GpuExecutor(cams, streams=1, max_frames=8)
    frames = [synth.generate_frame(synth.SceneSpec(c.width, c.height, c.handle.D,
                                                   synth.camera_for_size(c.width, c.height), seed=i))
              for i, c in [(1, cams[0]), (2, cams[1]), (3, cams[2]), (4, cams[0])]]
    reqs = [serving.Request(i, c, to_device(f), 0.0)
            for i, (c, f) in enumerate(zip([0, 1, 2, 0], frames))]
    announce("three height classes in one launch")
    assert len(ex.grouped(reqs)) == 1
    token = ex.launch(reqs)
    torch.cuda.synchronize()
    assert ex.finished(token)
    for r, f in zip(reqs, frames):
        assert_frames_equal(r.out.to_host(), oracle.frame(params[r.camera], f), str(r.rid))
