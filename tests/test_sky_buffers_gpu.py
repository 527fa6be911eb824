"""The work buffers a sky keeps between calls: what a call of many channels and
steps needed beyond the kept 1 GiB is given back when it ends, everything when
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
    s = make_sky(256, 460, np.linspace(50.0, 200.0, 401), 4, seed=3)
    edges = np.quantile(s.beta, np.linspace(0, 1, 9))
    sm = fgl.SkyModel.from_sky(s)                    # what the runtime takes at first use
    small = sm.chromatic(edges, np.arange(3)), sm.importance(np.arange(3), "sky")
    big = sm.chromatic(edges, np.arange(460))
    sm.close()
    start = free()
    sm = fgl.SkyModel.from_sky(s)
    sm.chromatic(edges, np.arange(3)), sm.importance(np.arange(3), "sky")
    made = free()
    # partial sums alone: about 100 items x 8 regions x 401 channels x 460 steps x 8 bytes, 1.2 GB
    assert np.array_equal(sm.chromatic(edges, np.arange(460)), big)
    kept = made - free()
    say(f"  kept after the large call: {kept / 2**20:.0f} MiB")
    assert kept <= 2**30
    again = sm.chromatic(edges, np.arange(3)), sm.importance(np.arange(3), "sky")
    assert all(np.array_equal(a, b) for a, b in zip(small, again))
    sm.close()
    assert start - free() < 64 * 2**20
