"""The path passes with costs in bytes against the oracle, bit for bit
(integer arithmetic): every layout of a line over lanes (4 to 256 disparities,
multiples of 8 and not), rows below and past a lane group's disparities, odd
sizes and remainders of a turn, calls of few lines (four directions in memory)
and of many (three, the last one fused with the selection), small calls on a
large handle, and the penalties on both sides of a byte."""

import numpy as np
import pytest

from oracle import sgm as osgm
import paper_1610_04124_amd as P
from paper_1610_04124_amd import binding as B
from gpu_helpers import announce, device

pytestmark = pytest.mark.gpu


def images(rng, n, H, W, shift=3):
    left = rng.integers(0, 256, (n, H, W), dtype=np.uint8)
    right = np.roll(left, -shift, axis=2)
    noise = rng.random(right.shape) < 0.2
    return left, np.where(noise, rng.integers(0, 256, right.shape, dtype=np.uint8), right)


def check(m, left, right, D, p1=10, p2=120):
    import torch
    got = m.compute(torch.from_numpy(left).to(device()), torch.from_numpy(right).to(device()))
    torch.cuda.synchronize()
    got = got.cpu().numpy().reshape(left.shape)
    H, W = left.shape[1:]
    seen = {}
    for i in range(len(left)):
        key = left[i].tobytes() + right[i].tobytes()
        if key not in seen:
            seen[key] = osgm.disparity(left[i], right[i], D, p1, p2)
        assert np.array_equal(got[i], seen[key]), i
    cl, cr = osgm.census(left[0]), osgm.census(right[0])
    three = sum(osgm.path(cl, cr, D, p1, p2, r).astype(np.int64) for r in (1, 2, 3))
    assert np.array_equal(m.debug(B.SGM_COSTS, W, H).astype(np.int64), three)


@pytest.mark.parametrize("W,H,D", [
    (1, 1, 4), (23, 6, 4), (57, 9, 32), (58, 13, 32), (64, 8, 36), (131, 7, 64), (90, 5, 72),
    (149, 11, 100), (152, 4, 128), (141, 9, 128), (150, 3, 136), (275, 9, 252), (281, 10, 256),
    (4203, 3, 32), (4100, 5, 64), (4099, 2, 128), (133, 70, 64)])
@pytest.mark.parametrize("many", [False, True])
def test_layouts_equal_oracle(W, H, D, many):
    # at most 17, 14 or 8 rows per compute unit are few
    lines = 256 * (17 if D <= 64 else 14 if D <= 128 else 8)
    n = lines // H + 2 if many else 3
    left, right = images(np.random.default_rng(W * D + H), 4, H, W)
    left, right = (np.tile(a, (n // 4 + 1, 1, 1))[:n] for a in (left, right))
    announce(f"sgm packed {W}x{H} D{D} x{n}")
    m = P.Sgm(W, H, D, max_frames=n)
    check(m, left, right, D)
    if many:
        # a small call on the same handle: few lines, its four planes within the three
        check(m, left[1:3], right[1:3], D)
        # few lines whose four planes don't fit go the other way
        check(m, left[:n - 4], right[:n - 4], D)
    m.close()


@pytest.mark.parametrize("p1,p2", [(0, 0), (0, 193), (193, 193), (5, 194), (194, 194), (0, 1000)])
@pytest.mark.parametrize("D", [60, 128])
def test_penalties_equal_oracle(p1, p2, D):
    left, right = images(np.random.default_rng(p1 + p2 + D), 2, 21, 151, shift=7)
    announce(f"sgm packed penalties {p1} {p2} D{D}")
    m = P.Sgm(151, 21, D, p1=p1, p2=p2, max_frames=2)
    check(m, left, right, D, p1, p2)
    m.close()
