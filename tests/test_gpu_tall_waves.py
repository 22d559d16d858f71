"""Tall columns shared by two and four waves against the oracle, bit for bit:
heights around slot counts (slots that the waves share unevenly), two and four
disparity chunks that end at different rows, invalid pixels, and shorter
frames in the same launch (a column that leaves half of the slots unused, one
that just needs more, one of a single slot)."""

import numpy as np
import pytest

import oracle
import synth
import paper_1610_04124_amd as P
from gpu_helpers import announce, assert_frames_equal, to_device

pytestmark = pytest.mark.gpu


def frame(H, W, D, rng, invalid):
    # disparities fall with the row; each 5-pixel column by its own slope
    v = np.arange(H - 1, -1, -1)[:, None]
    top = rng.integers(D // 8, D, W // 5).repeat(5)[None, :]
    d = np.floor(top * (1.0 - v / H) ** rng.uniform(0.5, 3.0, W // 5).repeat(5)[None, :])
    steps = rng.random((H, W // 5)) < 0.02
    d = d + np.cumsum(np.where(steps, rng.integers(-6, 7, steps.shape), 0), 0).repeat(5, axis=1)
    d = np.clip(d + rng.integers(-1, 2, d.shape), 0, D - 1).astype(np.float32)
    if invalid:
        d[rng.random(d.shape) < 0.2] = -1
        d[:, 5:10] = -1
    return d


@pytest.mark.parametrize("H", [577, 640, 705, 897, 1024])
@pytest.mark.parametrize("D", [128, 256])
@pytest.mark.parametrize("waves", [2, 4])
def test_tall_columns_equal_oracle(H, D, waves):
    check(H, D, waves)


@pytest.mark.parametrize("H", [321, 448, 512])
@pytest.mark.parametrize("D", [200, 256])
@pytest.mark.parametrize("waves", [1, 2, 4])
def test_four_chunks_equal_oracle(H, D, waves):
    """Five to eight slots, whose prior table drops chunks as the base rises."""
    check(H, D, waves)


def check(H, D, waves):
    import torch
    W, s = 20, 5
    rng = np.random.default_rng(H + D + waves)
    slots = (H + 63) // 64
    heights = [H, H, 64 * ((slots + 1) // 2 + 2), 64 * (slots // 2) - 7, 60]
    items, want = [], []
    for i, h in enumerate(heights):
        p = synth.make_params(camera=synth.camera_for_size(W, h), stixel_width=s,
                              max_disparity=D, max_width=W, max_height=h, flags=1)
        hd = P.Stixels(p)
        d = frame(h, W, D, rng, invalid=bool(i & 1))
        items.append((hd, to_device(d), hd.new_output(W, h)))
        want.append(oracle.frame(p, d))
    b = P.Batch(len(items), len(items) * (W // s), H, D)
    b.set_waves(waves)
    announce(f"tall columns H{H} D{D} waves {waves}")
    b.compute(items)
    torch.cuda.synchronize()
    assert b.waves() == waves
    for i, ((_, _, o), w) in enumerate(zip(items, want)):
        assert_frames_equal(o.to_host(), w, f"frame {i} of {heights[i]} rows")
