"""The recurrence without the second disparity chunk past the last row that
holds a disparity of it, against the oracle bit for bit: that row at the edges
of slots and columns, with and without invalid pixels (the table then starts
at disparity 0, else at the column's smallest), one, two and four waves per
column."""

import numpy as np
import pytest

import oracle
import synth
import paper_1610_04124_amd as P
from gpu_helpers import announce, assert_frames_equal, device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [64, 65, 200, 330])
@pytest.mark.parametrize("waves", [1, 2, 4])
@pytest.mark.parametrize("invalid", [False, True])
def test_last_row_of_the_second_chunk(H, waves, invalid):
    import torch
    W, s, D = 45, 5, 128
    rng = np.random.default_rng(H + invalid)
    cam = synth.camera_for_size(W, H)
    p = synth.make_params(camera=cam, stixel_width=s, max_disparity=D, max_width=W, max_height=H)
    # column c: rows up to last[c] (from the bottom) reach past disparity 64 + base
    last = [-1, 0, 1, 62, 63, 64, H // 2, H - 2, H - 1]
    base = 0 if invalid else 7
    d = np.empty((H, W), np.float32)
    for c, l in enumerate(last):
        v = np.arange(H - 1, -1, -1)[:, None]           # bottom-up row
        lo = rng.integers(base, base + 60, (H, s))
        hi = rng.integers(base + 56, base + 72, (H, s))
        d[:, c * s:(c + 1) * s] = np.where(v <= l, hi, lo)
        if 0 <= l < H:
            d[H - 1 - l, c * s:(c + 1) * s] = base + 64
    if invalid:
        d[rng.random((H, W)) < 0.3] = -1
    h = P.Stixels(p)
    out = h.new_output(W, H)
    b = P.Batch(1, W // s, H, D)
    cap = 4 if H > 192 else 2 if H > 64 else 1
    b.set_waves(waves)
    announce(f"second chunk H{H} waves {waves}")
    b.compute([(h, torch.from_numpy(d).to(device()), out)])
    torch.cuda.synchronize()
    assert b.waves() == min(waves, cap)
    want = oracle.frame(p, d)
    assert_frames_equal(out.to_host(), want, "batch")
    h.set_waves(min(waves, cap))
    out = h.compute(torch.from_numpy(d).to(device()))
    torch.cuda.synchronize()
    assert_frames_equal(out.to_host(), want, "frame")
    b.close()
    h.close()
