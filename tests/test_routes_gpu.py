"""Which kernels a call runs, on both sides of each line between two routes, by the
names of the launches that the profiler saw.  The tests that compare the routes'
results (test_thin_rows_gpu, test_chains_in_place_gpu, test_sky_lags_gpu) take their
shapes from these ranges."""
import re

import numpy as np
import pytest

import workload
from paper_2603_13196_amd import sampler as ns
from workload.sky import make_sky
from tests.gpu_util import lib, say

pytestmark = pytest.mark.gpu


def kernels(call):
    """Names of the library's kernels that `call` launches."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    found = {m.group(1) for e in p.events() for m in [re.search(r"fgl::(?:\(anonymous namespace\)::)?(k_\w+)", e.name)] if m}
    say(f"  {sorted(found)}")
    assert found
    return found


@pytest.mark.parametrize("N,F,T", [(1, 1, 1), (3, 2, 5), (4, 151, 1), (5, 64, 7), (8, 65, 30), (11, 33, 20), (12, 151, 2),
                                   (16, 151, 20), (20, 67, 9), (24, 30, 1), (32, 301, 1), (32, 63, 8)])
def test_small_thin_batches(N, F, T):
    import torch
    fgl = lib()
    freqs = np.linspace(50.0, 200.0, F) if F > 1 else np.array([120.0])
    w = workload.make(N, freqs, T, 2049, 500 + N, batch="mixed")
    m = fgl.Model.from_workload(w)
    th = torch.from_numpy(w.theta).cuda()
    out = torch.empty(2049, dtype=torch.float64, device="cuda")
    one, three = {"k_prep_thin64"}, {"k_prep", "k_thin64", "k_finalize"}
    m.loglike(w.theta[:300], "mixed"), m.loglike_device(th), m.loglike_device(th[:300].contiguous())
    assert kernels(lambda: m.loglike(w.theta[:300], "mixed")) == one
    rows = th[:300].contiguous()
    # two turns over the channels of 32 regions cost more than the two launches
    assert kernels(lambda: m.loglike_device(rows, out[:300])) == (three if (N, F) == (32, 301) else one)
    assert kernels(lambda: m.loglike_device_noalloc(rows, out[:300])) == (three if (N, F) == (32, 301) else one)
    assert kernels(lambda: m.loglike_device(th, out)) == three          # past 2048 rows
    assert kernels(lambda: fgl.fgl_loglike_batch_device(             # results over the rows
        m.handle, rows.data_ptr(), 300, rows.data_ptr(), "mixed",
        torch.cuda.current_stream().cuda_stream)) == three
    m.close()


@pytest.mark.parametrize("N,F,T,n,steps,inside", [
    (1, 1, 1, 3, 5, True), (4, 64, 64, 17, 4, True), (10, 151, 1, 70, 12, True), (16, 301, 20, 20, 3, True),
    (32, 190, 8, 16, 3, True), (8, 701, 2, 12, 4, True), (4, 301, 64, 300, 2, False), (8, 301, 40, 1000, 2, False),
    (24, 301, 60, 16, 2, False),
])
def test_chain_rounds(N, F, T, n, steps, inside):
    fgl = lib()
    freqs = np.linspace(50.0, 200.0, F) if F > 1 else np.array([120.0])
    w = workload.make(N, freqs, T, 8, 4000 + N + T)
    m = fgl.Model.from_workload(w)
    lo, hi = ns.foreground_box(N)
    rng = np.random.Generator(np.random.PCG64(n))
    x = np.clip((lo + hi) / 2 + 0.05 * (hi - lo) * rng.standard_normal((n, lo.size)), lo, hi)
    lx = m.loglike(ns.to_theta(x), "mixed")
    chol = np.diag(0.01 * (hi - lo))
    eng = fgl.Chains(m, n, lo, hi, seed=5)
    call = lambda: eng.run(x, lx, float(lx.min()) - 1.0, chol, steps, "mixed")
    call()
    got = kernels(call)
    assert ("k_chain_run" in got) == inside and ("k_chain_step" in got) == (not inside)
    m.kernel_timing(True)
    timed = kernels(call)
    m.kernel_timing(False)
    assert "k_chain_step" in timed and "k_chain_run" not in timed
    eng.close()
    m.close()


@pytest.mark.parametrize("nlon,T,step,grid", [
    (340, 3, 1, True), (339, 3, 1, False), (240, 50, 2, True), (240, 49, 2, False), (640, 96, 5, True),
    (512, 6, 67, False), (700, 600, 1, True), (5, 4, 1, False),
])
def test_importance_maps(nlon, T, step, grid):
    fgl = lib()
    s = make_sky(4, nlon, np.linspace(50.0, 200.0, 5), T, seed=nlon)
    sm = fgl.SkyModel.from_sky(s)
    shifts = (np.arange(T) * step % nlon).astype(np.int32)
    if step == 67:
        shifts = np.array([0, 3, 50, 111, 300, 511], dtype=np.int32)      # scattered
    got = kernels(lambda: sm.importance(shifts, "sky"))
    assert ("k_lag_imp" in got) == grid and ("k_sky_importance" in got) == (not grid)
    sm.close()
