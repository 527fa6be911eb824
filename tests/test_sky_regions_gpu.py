"""Grouping of pixels by region on the device: edges on pixel values, repeated
and one-sided edges, more regions than a workgroup has threads, regions without
pixels, rings and columns that no step sees through the beam (left out) and a
beam that is zero everywhere, against the FP64 oracle; calls of different sizes
on one sky, from several threads."""
import threading

import numpy as np
import pytest

from oracle import regions
from workload.sky import Sky, make_sky
from tests.gpu_util import lib, say

pytestmark = pytest.mark.gpu


def _check(sm, s, edges, shifts):
    sub = Sky(s.omega, s.t_ex, s.beta, s.beam, s.horizon, s.freqs, np.asarray(shifts, np.int32))
    got = sm.chromatic(edges, sub.shifts)
    want = regions.chromatic(sub, regions.masks(s.beta, edges), len(edges) - 1)
    # sums of at most nlat nlon terms of one sign, a rounding or two per term
    scale = np.abs(want).max() if want.size else 0.0
    tol = (s.nlat * s.nlon + 8) * 2.0 ** -52 * np.maximum(np.abs(want), 1e-300)
    d = np.abs(got - want)
    say(f"  N{len(edges) - 1} T{len(shifts)}: max|d|={d.max():.2e} of scale {scale:.2e}")
    assert np.all(d <= tol)


def _sky(nlat, nlon, F, seed, dark=False):
    s = make_sky(nlat, nlon, np.linspace(50.0, 200.0, F), 4, seed=seed)
    rng = np.random.Generator(np.random.PCG64(seed))
    beam = s.beam * (rng.random(s.beam.shape) > 0.3)
    beam[:, nlat // 3] = 0.0                       # a ring without a beam
    beam[:, :, nlon // 2:] *= rng.random((F, nlat, nlon - nlon // 2)) > 0.9
    if dark:
        beam[:] = 0.0
    return Sky(s.omega, s.t_ex, s.beta, beam.astype(np.float32), s.horizon, s.freqs, s.shifts)


@pytest.mark.parametrize("nlat,nlon,F", [(5, 16, 3), (12, 70, 5), (7, 257, 4), (3, 1, 2), (4, 530, 2)])
def test_region_edges(nlat, nlon, F):
    fgl = lib()
    s = _sky(nlat, nlon, F, nlat * 100 + nlon)
    say(f"sky {nlat}x{nlon} F={F}")
    sm = fgl.SkyModel.from_sky(s)
    b = np.sort(s.beta.ravel())
    lo, hi, mid = b[0], b[-1], b[b.size // 2]
    for edges in ([lo, hi], [lo, mid, hi], [lo, mid, mid, hi], [mid, mid], [lo - 1, lo], [hi, hi + 1],
                  [hi + 1, hi + 2], np.linspace(lo, hi, 10), np.linspace(lo - 0.1, hi + 0.1, 301),
                  np.linspace(mid - 0.01, mid + 0.01, 1025)):
        for shifts in ([0], [nlon - 1], list(np.arange(5) % nlon)):
            _check(sm, s, np.asarray(edges, dtype=np.float64), shifts)
    sm.close()


def test_dark_beam_and_calls_in_turn():
    fgl = lib()
    s = _sky(6, 40, 3, 11, dark=True)
    sm = fgl.SkyModel.from_sky(s)
    assert not np.any(sm.chromatic([1.0, 2.6, 4.0], [0, 3, 7]))
    sm.close()
    s = _sky(9, 60, 5, 12)
    sm = fgl.SkyModel.from_sky(s)
    e = np.quantile(s.beta, np.linspace(0, 1, 8))
    big = np.quantile(s.beta, np.linspace(0, 1, 41))
    want = {}
    for k in range(3):                             # buffers that grow, then serve less
        for name, (edges, n) in {"a": (e, 5), "b": (big, 60), "c": (e[:3], 1)}.items():
            got = sm.chromatic(edges, np.arange(n)), sm.importance(np.arange(n), "sky")
            if name in want:
                assert all(np.array_equal(x, y) for x, y in zip(got, want[name])), name
            want[name] = got
    bad = []

    def work(name, edges, n):
        for _ in range(5):
            got = sm.chromatic(edges, np.arange(n)), sm.importance(np.arange(n), "sky")
            if not all(np.array_equal(x, y) for x, y in zip(got, want[name])):
                bad.append(name)

    ts = [threading.Thread(target=work, args=a) for a in (("a", e, 5), ("b", big, 60), ("c", e[:3], 1))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
    sm.close()
