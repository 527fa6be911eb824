"""Small batches of thin models, evaluated in one launch, against the rows of a
batch large enough for the three launches, bit for bit: batch sizes around the
rows a workgroup takes, every compiled region count, channel counts around the
group size, amplitude masks, no 21-cm term, invalid rows, from host and device
memory, without allocation, and with results written over the rows."""
import numpy as np
import pytest

import workload
from tests.gpu_util import lib, say

pytestmark = pytest.mark.gpu


def _same(fgl, w, flags=0, sizes=(1, 3, 4, 5, 17, 300)):
    import torch
    m = fgl.Model.from_workload(w, flags=flags)
    assert m.form == "thin"
    theta = w.theta.copy() if not flags & fgl.FGL_NO_21CM else \
        np.ascontiguousarray(np.delete(w.theta, [w.P - 4, w.P - 3, w.P - 2], axis=1))
    P = theta.shape[1]
    theta[2, 0], theta[7, P - 1], theta[11, 0] = np.nan, -1.0, 65.0
    if not flags & fgl.FGL_NO_21CM:
        theta[13, P - 2] = 0.0
    reps = int(3e8 / (theta.shape[0] * w.F * 16)) + 2        # past the one-launch line
    want = m.loglike(np.tile(theta, (reps, 1)), "mixed")[:theta.shape[0]]
    assert np.array_equal(np.isneginf(want[:14]), np.isin(np.arange(14),
                          [2, 7, 11] if flags & fgl.FGL_NO_21CM else [2, 7, 11, 13]))
    for B in sizes:
        B = min(B, theta.shape[0])
        for prec in ("mixed", "fp64"):
            assert np.array_equal(m.loglike(theta[:B], prec), want[:B]), (B, prec)
        th = torch.from_numpy(theta[:B].copy()).cuda()
        assert np.array_equal(m.loglike_device(th).cpu().numpy(), want[:B]), B
        out = torch.empty(B, dtype=torch.float64, device="cuda")
        assert np.array_equal(m.loglike_device_noalloc(th, out).cpu().numpy(), want[:B]), B
        over = th.view(-1)[:B]                               # results over the rows
        fgl.fgl_loglike_batch_device(m.handle, th.data_ptr(), B, over.data_ptr(), "mixed",
                                     torch.cuda.current_stream().cuda_stream)
        assert np.array_equal(over.cpu().numpy(), want[:B]), B
    m.close()


@pytest.mark.parametrize("N,F,T", [(1, 1, 1), (3, 2, 5), (4, 151, 1), (5, 64, 7), (8, 65, 30),
                                   (11, 33, 20), (12, 151, 2), (16, 151, 20), (20, 67, 9),
                                   (24, 30, 1), (32, 301, 1), (32, 63, 8)])
def test_one_launch_equals_three(N, F, T):
    say(f"N={N} F={F} T={T}")
    fgl = lib()
    freqs = np.linspace(50.0, 200.0, F) if F > 1 else np.array([120.0])
    _same(fgl, workload.make(N, freqs, T, 300, 500 + N + F + T, batch="mixed"))


def test_one_launch_batch_sizes():
    w = workload.make(4, np.linspace(50.0, 200.0, 31), 1, 5000, 77, batch="mixed")
    _same(lib(), w, sizes=(255, 256, 1000, 1023, 1024, 1025, 2047, 2048, 2049, 4999, 5000))


def test_one_launch_masks_and_without_21cm():
    fgl = lib()
    _same(fgl, workload.make_masks(3, 4, np.linspace(50.0, 200.0, 45), 3, 300, 5, batch="mixed"))
    _same(fgl, workload.make(7, np.linspace(50.0, 200.0, 45), 3, 300, 6, batch="mixed"),
          flags=fgl.FGL_NO_21CM)
