"""Importance maps over many patterns of shifts: evenly spaced steps of every
spacing (the lag-grid kernels, whole and ragged blocks of columns and lags, one
and several residue classes, wrapped and repeated steps), scattered steps on and
off that grid, ragged and empty horizons, against the FP64 oracle."""
import numpy as np
import pytest

from oracle import regions
from workload.sky import Sky, make_sky
from tests.gpu_util import lib, say

pytestmark = pytest.mark.gpu


def _shifts(kind, nlon, T):
    rng = np.random.Generator(np.random.PCG64(nlon + T))
    if kind == "scattered":
        return rng.integers(0, nlon, size=T)
    if kind == "near":                       # most of a short run of lags, out of order
        return rng.permutation(np.arange(2 * T) % nlon)[:T]
    if kind == "zero":
        return np.zeros(T, dtype=np.int64)
    return (np.arange(T) * int(kind)) % nlon


@pytest.mark.parametrize("kind,nlat,nlon,F,T", [
    ("1", 9, 64, 5, 16), ("1", 7, 65, 4, 17), ("1", 5, 48, 9, 48), ("1", 6, 33, 3, 90),
    ("1", 4, 300, 5, 140), ("1", 3, 700, 2, 600), ("2", 6, 97, 6, 30), ("3", 6, 64, 5, 12),
    ("5", 5, 128, 4, 96), ("7", 6, 50, 3, 8), ("21", 4, 512, 3, 4), ("near", 6, 120, 5, 20),
    ("scattered", 6, 40, 5, 24), ("scattered", 5, 512, 4, 6), ("zero", 4, 20, 3, 5),
    ("1", 4, 1, 2, 1), ("1", 3, 17, 1, 1),
    # rings wide enough for the grid kernels whatever the steps, and the columns
    # and columns times steps on both sides of that line
    ("1", 5, 400, 9, 48), ("2", 4, 341, 6, 30), ("5", 5, 640, 4, 96), ("7", 6, 350, 3, 8),
    ("near", 6, 420, 5, 20), ("scattered", 5, 400, 5, 24), ("zero", 4, 340, 3, 5),
    ("1", 3, 357, 1, 1), ("3", 6, 339, 5, 17), ("2", 5, 240, 4, 50), ("2", 5, 240, 4, 49),
])
def test_importance_over_shift_patterns(kind, nlat, nlon, F, T):
    fgl = lib()
    s = make_sky(nlat, nlon, np.linspace(50.0, 200.0, F), T, seed=nlon + T)
    rng = np.random.Generator(np.random.PCG64(nlat * nlon))
    shifts = _shifts(kind, nlon, T).astype(np.int32)
    hor = s.horizon.copy()
    if nlon > 30:                            # holes, single columns and an empty ring
        hor[:, rng.integers(0, nlon, size=nlon // 7)] ^= 1
        hor[nlat // 2] = 0
    hor[0, 0] = hor[-1, -1] = 1
    beam = (s.beam + 0.01).astype(np.float32)
    s = Sky(s.omega, s.t_ex, s.beta, beam, hor, s.freqs, shifts)
    sm = fgl.SkyModel.from_sky(s)
    for sch in regions.SCHEMES:
        got = sm.importance(shifts, sch)
        want = regions.importance(s, sch)
        # both are sums of positive FP64 terms, the longest of nlat nlon + F T of
        # them, and a few roundings per term
        tol = (nlat * nlon + F * T + 32) * 2.0 ** -52
        d = np.abs(got - want) / np.where(want > 0, want, 1.0)
        say(f"  {kind} {nlat}x{nlon} F{F} T{T} {sch}: {d.max():.2e} of {tol:.2e}")
        assert np.all(d <= tol)
    sm.close()
