"""FrameOutput on the CPU: four arrays in one allocation, and the sizes it takes."""

import numpy as np
import pytest
import torch

from paper_1610_04124_amd.binding import FrameOutput


@pytest.mark.parametrize("ncols,cap", [(0, 5), (5, 0), (1, 1), (3, 7), (np.int64(204), 440)])
def test_arrays(ncols, cap):
    o = FrameOutput(ncols, cap, torch.device("cpu"))
    for name, shape, dtype in [("counts", (ncols,), torch.int32), ("total", (ncols,), torch.float32),
                               ("records", (ncols, cap, 3), torch.int32),
                               ("overflow", (ncols,), torch.uint8)]:
        t = getattr(o, name)
        assert tuple(t.shape) == shape and t.dtype == dtype and t.is_contiguous()
        assert int((t != 0).sum()) == 0
    # writing one leaves the others alone
    o.counts.fill_(-1)
    o.overflow.fill_(9)
    assert int((o.records != 0).sum()) == 0 and int((o.total != 0).sum()) == 0


@pytest.mark.parametrize("ncols,cap,error", [
    (-1, 5, RuntimeError), (5, -1, RuntimeError), (-3, -3, RuntimeError), (3.0, 4, TypeError),
    (3, 4.5, TypeError), ("3", 4, TypeError),
])
def test_sizes_that_are_none(ncols, cap, error):
    with pytest.raises(error):
        FrameOutput(ncols, cap, torch.device("cpu"))
