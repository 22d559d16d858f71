"""Columns spread over workgroups: how many waves a workgroup has and how many
workgroups share a compute unit follow from the LDS a column of that height
takes, on every entry point that spreads columns, and the results equal the CPU
oracle bit for bit on both sides of each line."""

import numpy as np
import pytest

import oracle
import paper_1610_04124_amd as P
from gpu_helpers import announce, assert_frames_equal, device, to_device
from test_gpu_chain import frame_and_params

pytestmark = pytest.mark.gpu

COLS, TILE = 1100, 44


def wide_frame(H, D, flags=0):
    """A frame of COLS one-pixel columns that repeat TILE of them, and the oracle's tile."""
    p, disp = frame_and_params(H, D, "columns", s=1, cols=TILE)
    disp = disp[:, :TILE]
    p = dict(p, max_width=COLS, flags=flags)
    return p, np.tile(disp, (1, COLS // TILE)), oracle.frame(p, disp)


def assert_tiles_equal(out, ref, label):
    host = out.to_host()
    for i in range(0, COLS, TILE):
        assert_frames_equal({k: v[i:i + TILE] for k, v in host.items()}, ref, f"{label} from {i}")


# waves of a workgroup and workgroups of a compute unit (256 of them: more
# columns than that, so a column has no compute unit to itself by their number)
@pytest.mark.parametrize("H,waves,per_cu", [
    (33, 4, 4), (64, 4, 4), (65, 6, 2), (129, 8, 2), (440, 8, 2), (513, 8, 2), (888, 8, 2),
    (889, 16, 1), (1024, 16, 1),
])
def test_batch_fills_what_lds_admits(H, waves, per_cu):
    import torch
    announce(f"resident workgroups of a batch, H={H}")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    p, disp, ref = wide_frame(H, 16, flags=1)
    h = P.Stixels(p)
    out = h.new_output(COLS, H)
    b = P.Batch(1, COLS, H, 16)
    b.compute([(h, to_device(disp), out)])
    torch.cuda.synchronize()
    assert_tiles_equal(out, ref, f"batch {H}")
    assert b.waves() == waves
    assert b.info()[0] == min(per_cu * cus, COLS)
    b.close()
    h.close()


@pytest.mark.parametrize("H", [64, 888, 889, 890, 895, 896, 1024])
def test_frames_on_both_sides_of_the_line(H):
    """One launch (a frame's own variables leave room for one row more), the
    recurrence over tables in memory, and the entry that allocates nothing."""
    import torch
    announce(f"frames of {COLS} columns, H={H}")
    p, disp, ref = wide_frame(H, 16)
    h = P.Stixels(p)
    frame = to_device(disp)
    for label in ("one launch", "online costs", "noalloc"):
        out = h.new_output(COLS, H)
        out.counts.fill_(-7)
        h.set_object_lut(1 if label == "online costs" else 0)
        if label == "noalloc":
            h.compute_noalloc(frame, out)
        else:
            h.compute(frame, out)
        torch.cuda.synchronize()
        assert_tiles_equal(out, ref, f"{label} {H}")
    h.close()


@pytest.mark.parametrize("H,D,per_cu", [
    (64, 64, 9), (65, 64, 6), (128, 128, 6), (320, 128, 6), (128, 256, 7), (320, 256, 7),
    (321, 64, 7), (384, 128, 7), (384, 256, 9), (385, 64, 10), (448, 128, 10), (448, 256, 18),
    (449, 64, 18), (512, 128, 18), (512, 256, 28),
])
def test_line_between_spread_and_one_wave(H, D, per_cu):
    """An automatic batch spreads its columns up to so many per compute unit."""
    import torch
    announce(f"line of automatic batches, H={H} D={D}")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    p, disp = frame_and_params(H, D, "columns", s=1, cols=TILE)
    ref = oracle.frame(p, disp[:, :TILE])
    cols = per_cu * cus + 1
    h = P.Stixels(dict(p, max_width=cols, flags=1))
    frame = to_device(disp[:, :TILE]).repeat(1, -(-cols // TILE))
    b = P.Batch(1, cols, H, D)
    for n, spread in ((cols - 1, True), (cols, False)):
        o = P.FrameOutput(n, H, device())
        b.compute([(h, frame[:, :n].contiguous(), o)])
        torch.cuda.synchronize()
        assert (b.waves() > 1) == spread
        host = o.to_host()
        for i in range(0, n // TILE * TILE, 8 * TILE):
            assert_frames_equal({k: v[i:i + TILE] for k, v in host.items()}, ref, f"{n} from {i}")
    b.close()
    h.close()
