"""The staged path's recurrence spread over a workgroup (the default: neither
waves nor table placement set) against the CPU oracle, bit for bit, at the
sizes where its parts meet: groups of 8 steps run in pairs, slots and windows
of 64 rows, bounds in blocks of 32 rows, one to sixteen slots."""

import numpy as np
import pytest

import oracle
import synth
import paper_1610_04124_amd as P
from gpu_helpers import announce, assert_frames_equal, gpu_frame

pytestmark = pytest.mark.gpu


def frame_and_params(H, D, kind, s=3, cols=12, sub=0):
    W = s * cols + 1
    rng = np.random.default_rng(1000 * H + D)
    cam = dict(synth.CAMERA_1024x440, horizon_row=float(H * 37 // 100))
    p = synth.make_params(camera=cam, stixel_width=s, max_disparity=D, max_width=W, max_height=H,
                          subpixel_log2=sub)
    if kind == "columns":                  # every kind of pixel, in strips
        return p, synth.random_columns_frame(H + D, W, H, D)
    disp = np.empty((H, W), np.float32)
    if kind == "one object":               # one disparity: no group can be skipped, ties all over
        disp[:] = float(D // 3)
    elif kind == "object steps":           # long objects, means that rise and fall by one
        disp[:] = D // 4 + (np.arange(H)[:, None] // 97) % 2
        disp[rng.random((H, W)) < 0.3] = -1.0
    elif kind == "noise":
        disp[:] = rng.uniform(0, D - 1, (H, W))
    else:                                  # ground ramp into sky
        disp[:] = np.maximum(0.25 * (np.arange(H) - cam["horizon_row"]), 0.0)[:, None]
        disp += rng.normal(0, 0.8, (H, W))
        np.clip(disp, 0, D - 1, out=disp)
    return p, disp


@pytest.mark.parametrize("H,D,kind", [
    (1, 16, "columns"), (7, 16, "columns"), (8, 16, "noise"), (17, 64, "columns"),
    (63, 64, "one object"), (64, 64, "columns"), (65, 64, "object steps"),
    (127, 128, "ramp"), (128, 128, "one object"), (129, 128, "columns"),
    (191, 128, "object steps"), (193, 200, "columns"), (257, 128, "one object"),
    (440, 128, "ramp"), (449, 128, "object steps"), (511, 256, "columns"),
    (513, 256, "one object"), (640, 96, "noise"), (705, 128, "object steps"),
    (880, 256, "ramp"), (897, 256, "one object"), (961, 256, "columns"),
    (1024, 256, "object steps"),
])
def test_chain_edges(H, D, kind):
    announce(f"chain H={H} D={D} {kind}")
    p, disp = frame_and_params(H, D, kind)
    h = P.Stixels(p)
    assert_frames_equal(gpu_frame(h, disp), oracle.frame(p, disp), f"{kind} {H}")
    h.close()


@pytest.mark.parametrize("cols", [255, 256, 257, 300])
def test_chain_workgroup_sizes(cols):
    """Sixteen waves a column up to the compute unit count, eight above it."""
    announce(f"chain columns {cols}")
    p, disp = frame_and_params(200, 64, "object steps", s=2, cols=cols)
    h = P.Stixels(p)
    assert_frames_equal(gpu_frame(h, disp), oracle.frame(p, disp), f"{cols} columns")
    h.close()


def test_chain_priors_and_capacity():
    """Large ordering tolerance, free transitions (ties between classes), more
    than 64 stixels a column, sub-pixel bins and a short output."""
    announce("chain priors")
    p, disp = frame_and_params(300, 64, "noise", sub=1)
    p["model"].update(bic_cost=0.0, ordering_tol_px=1 << 20, ordering_cost=0.0,
                      trans_cost=[[0.0] * 3 for _ in range(3)], first_cost=[0.0] * 3)
    h = P.Stixels(p)
    ref = oracle.frame(p, disp)
    assert int(ref["counts"].max()) > 64
    assert_frames_equal(gpu_frame(h, disp), ref, "free transitions")
    assert_frames_equal(gpu_frame(h, disp, capacity=5), oracle.frame(p, disp, cap=5), "capacity")
    h.close()


@pytest.mark.parametrize("heights", [(64, 65, 440), (1024, 7, 513, 128), (512, 300)])
def test_chain_batch_mixed(heights):
    """Frames of several heights, disparity ranges and column counts in one
    automatic launch (more columns than workgroups, so that workgroups go from
    one column to another of a different height), captured and replayed."""
    import torch
    announce(f"chain batch {heights}")
    st = torch.cuda.Stream()
    items, refs = [], []
    for i, H in enumerate(heights):
        p, disp = frame_and_params(H, (64, 128, 256)[i % 3], ("columns", "object steps")[i % 2],
                                   s=2, cols=250)
        h = P.Stixels(dict(p, flags=1))
        t = torch.from_numpy(np.ascontiguousarray(disp)).cuda()
        items.append((h, t, h.new_output(disp.shape[1], H)))
        refs.append(oracle.frame(p, disp))
    torch.cuda.synchronize()
    b = P.Batch(len(items), 250 * len(items), max(heights), 256)
    b.capture(items, st)
    assert b.waves() > 4                  # a workgroup per column
    for _ in range(3):
        for _, _, o in items:
            o.counts.zero_()
            o.records.zero_()
        torch.cuda.synchronize()
        b.replay(st)
        torch.cuda.synchronize()
        for (_, _, o), ref, H in zip(items, refs, heights):
            assert_frames_equal(o.to_host(), ref, f"batch {H}")
    b.close()
