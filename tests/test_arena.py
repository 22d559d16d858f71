"""Table space of frames whose columns do not all fit the fixed workspace of
stixels_compute_noalloc: places handed out never overlap, also after more
requests than a 32-bit count of them could hold (CPU), and such a frame equals
the oracle bit for bit (GPU)."""

import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1610_04124_amd", "csrc")
ROOM = (64 << 20) // 16                       # 16-byte units of the workspace
TALLEST = 256 * ((1024 + 10) // 4)            # units of a table of 1024 rows and 256 bins


@pytest.fixture(scope="module")
def sim(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("arena") / "sim")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", CSRC,
                    os.path.join(HERE, "arena_sim.cpp"), "-o", exe], check=True)
    return lambda *a: tuple(map(int, subprocess.run([exe, *map(str, a)], check=True,
                                                    capture_output=True, text=True).stdout.split()))


@pytest.mark.parametrize("columns", [63, 64, 1024, 65_000, 66_000, 200_000])
def test_places_do_not_overlap(sim, columns):
    given, bad = sim(ROOM, TALLEST, columns)
    assert (given, bad) == (min(columns, ROOM // TALLEST), 0)


def test_small_requests_fill_the_space(sim):
    assert sim(1000, 7, 100_000) == (1000 // 7, 0)
    assert sim(6, 7, 10) == (0, 0)


@pytest.mark.gpu
def test_more_columns_than_a_count_of_requests_holds():
    """90,000 columns of 1024 rows that hold all of 256 bins: 63 tables fit the
    workspace."""
    import torch
    import oracle
    import synth
    import paper_1610_04124_amd as P
    from gpu_helpers import announce, assert_frames_equal, device, to_device

    W, H, D, tile = 90_000, 1024, 256, 50
    p = synth.make_params(camera=dict(synth.CAMERA_1024x440, horizon_row=400.0), stixel_width=1,
                          max_disparity=D, max_width=W, max_height=H, max_stixels_per_column=64,
                          flags=1)
    disp = synth.random_columns_frame(5, tile, H, D)
    disp[300], disp[700] = 0.0, D - 1.0
    ref = oracle.frame(p, disp, cap=64)
    h = P.Stixels(p)
    out = P.FrameOutput(W, 64, device())
    announce(f"noalloc {W}x{H} D={D} s=1")
    h.compute_noalloc(to_device(disp).repeat(1, W // tile), out)
    torch.cuda.synchronize()
    whole = {k: getattr(out, k).view(W // tile, tile, *getattr(out, k).shape[1:])
             for k in ("counts", "records", "total", "overflow")}
    for t in whole.values():                  # every repetition equals the first
        assert bool((t == t[:1]).all())
    first = P.FrameOutput(tile, 64, torch.device("cpu"))
    for k, t in whole.items():
        setattr(first, k, t[0].cpu())
    assert_frames_equal(first.to_host(), ref, "the first columns")
    h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("W,H,D", [
    (2000, 64, 128), (2000, 96, 128), (2000, 97, 128), (4300, 64, 256), (4300, 65, 256),
    (4000, 64, 256), (5000, 16, 256), (1000, 32, 256),
])
def test_frames_on_both_sides_of_the_line(W, H, D):
    """Columns spread over workgroups or a wave each, by rows, bins and columns."""
    import torch
    import oracle
    import synth
    import paper_1610_04124_amd as P
    from gpu_helpers import announce, assert_frames_equal, device, to_device

    tile = 50
    p = synth.make_params(camera=dict(synth.CAMERA_1024x440, horizon_row=float(H // 3)),
                          stixel_width=1, max_disparity=D, max_width=W, max_height=H, flags=1)
    disp = synth.random_columns_frame(W + H, tile, H, D)
    ref = oracle.frame(p, disp)
    h = P.Stixels(p)
    frame = to_device(disp).repeat(1, W // tile)
    announce(f"noalloc {W}x{H} D={D} s=1")
    for _ in range(2):                        # the workspace holds the last call's tables
        out = P.FrameOutput(W, H, device())
        out.counts.fill_(-7)
        h.compute_noalloc(frame, out)
        torch.cuda.synchronize()
        host = out.to_host()
        for i in range(0, W, tile):
            assert_frames_equal({k: v[i:i + tile] for k, v in host.items()}, ref, f"from {i}")
    h.close()
