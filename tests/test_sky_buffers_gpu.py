"""The work buffers a sky keeps between calls: what a call of many channels and
steps needed beyond the kept 512 MiB is given back when it ends, everything when
the sky is closed, and calls after it return what they did."""
import numpy as np
import pytest

from workload.sky import make_sky
from tests.gpu_util import lib, say

pytestmark = pytest.mark.gpu


def test_kept_buffers_are_bounded():
    import torch
    fgl = lib()
    torch.cuda.set_device(0)
    free = lambda: (torch.cuda.synchronize(), torch.cuda.mem_get_info()[0])[1]
    s = make_sky(256, 400, np.linspace(50.0, 200.0, 200), 4, seed=3)
    edges = np.quantile(s.beta, np.linspace(0, 1, 9))
    start = free()
    sm = fgl.SkyModel.from_sky(s)
    small = sm.chromatic(edges, np.arange(3)), sm.importance(np.arange(3), "sky")
    made = free()
    # partial sums alone: 128 items x 8 regions x 200 channels x 400 steps x 8 bytes, 655 MB
    big = sm.chromatic(edges, np.arange(400))
    kept = made - free()
    say(f"  kept after the large call: {kept / 2**20:.0f} MiB")
    assert kept <= 512 * 2**20
    again = sm.chromatic(edges, np.arange(3)), sm.importance(np.arange(3), "sky")
    assert all(np.array_equal(a, b) for a, b in zip(small, again))
    assert np.array_equal(sm.chromatic(edges, np.arange(400)), big)
    sm.close()
    assert start - free() < 64 * 2**20
