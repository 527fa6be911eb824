"""Importance calls that are refused, on rings wide enough for the lag-grid
kernels and on narrow ones: a weight that integrates to zero at a step names that
step's channel and leaves the caller's map as it was."""
import ctypes

import numpy as np
import pytest

from workload.sky import Sky, make_sky
from tests.gpu_util import lib, say

pytestmark = pytest.mark.gpu


def _importance(fgl, sm, shifts, scheme, out):
    sh = np.ascontiguousarray(shifts, dtype=np.int32)
    return fgl._lib.fgl_sky_importance(sm.handle, sh.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), sh.size,
                                       fgl.WEIGHTS[scheme], out.ctypes.data_as(fgl._dp))


@pytest.mark.parametrize("nlon,T", [(400, 12), (60, 12)])
def test_refused_maps_are_left_alone(nlon, T):
    fgl = lib()
    s = make_sky(6, nlon, np.linspace(50.0, 200.0, 7), T, seed=nlon)
    beam = np.ascontiguousarray(s.beam + 0.01, dtype=np.float32)
    beam[5] = 0.0                                    # one channel sees nothing
    hor = np.ones_like(s.horizon)
    sm = fgl.SkyModel.from_sky(Sky(s.omega, s.t_ex, s.beta, beam, hor, s.freqs, s.shifts))
    out = np.full((6, nlon), 7.25)
    rc = _importance(fgl, sm, np.arange(T), "beam", out)
    say(f"  {nlon} columns: {rc} {fgl.fgl_last_error()}")
    assert rc == fgl.FGL_EINVAL and "channel 5, step 0 integrates to 0" in fgl.fgl_last_error()
    assert np.all(out == 7.25)
    assert _importance(fgl, sm, np.arange(T), "sky", out) == fgl.FGL_OK
    assert np.all(np.isfinite(out)) and not np.any(out == 7.25)
    sm.close()


@pytest.mark.parametrize("nlon", [400, 60])
def test_weights_past_the_range(nlon):
    """A pixel below the horizon whose T_sky overflows: its products with the zero
    beam are NaN, so the map is refused and K of its region is NaN, whichever kernels
    a call takes; products are left out only where they are zero."""
    fgl = lib()
    s = make_sky(6, nlon, np.linspace(50.0, 200.0, 7), 12, seed=nlon)
    beam = np.ascontiguousarray(s.beam + 0.01, dtype=np.float32)
    hor = np.ones_like(s.horizon)
    hor[:, nlon // 2:] = 0                           # and nothing seen there
    beam[:, :, nlon // 2:] = 0.0
    t_ex, beta = s.t_ex.copy(), s.beta.copy()
    beta[2, nlon - 2], t_ex[2, nlon - 2] = 64.0, 1e300
    omega = s.omega * 1e16
    sm = fgl.SkyModel.from_sky(Sky(omega, t_ex, beta, beam, hor, s.freqs, s.shifts))
    out = np.full((6, nlon), 7.25)
    rc = _importance(fgl, sm, np.arange(12), "sky", out)
    say(f"  {nlon} columns: {rc} {fgl.fgl_last_error()}")
    assert rc == fgl.FGL_EINVAL and "integrates to" in fgl.fgl_last_error()
    assert np.all(out == 7.25)
    K = sm.chromatic([0.0, 10.0, 65.0], np.arange(12))
    assert np.all(np.isnan(K[1])) and np.all(np.isfinite(K[0]))
    assert _importance(fgl, sm, np.arange(12), "horizon", out) == fgl.FGL_OK
    assert np.all(np.isfinite(out))
    sm.close()
