"""The mixed kernel over its region slots and row groups: region counts around
every slot count (4, 8, 12, 16 per lane and chunk), chunk and tile edge, in the
projected form (last row tile of one to thirty-two rows, chunks left out of later
tiles), and time bins around every eighth row in the direct form, with and
without amplitude masks, against the FP64 oracle at the mixed bar."""
import numpy as np
import pytest

import oracle
import workload
from tests.gpu_util import check, lib, say

pytestmark = pytest.mark.gpu
FREQS = np.linspace(50.0, 200.0, 7)


def _run(w, form, flags=0):
    fgl = lib()
    ref = oracle.load().loglike_w(w)
    m = fgl.Model.from_workload(w, flags=flags)
    assert m.form == form
    got = m.loglike(w.theta, "mixed")
    check(got, ref, "mixed", f"{form} N{w.N} T{w.T} a{w.n_alpha}")
    # every tile gives the same bits
    for waves in (4, 8):
        for occ in (2, 3):
            for chans in (1, 2, 4, 8):
                try:
                    m.set_tile(w.B, "mixed", waves, chans, occ)
                except fgl.FGLError:
                    continue
                assert np.array_equal(m.loglike(w.theta, "mixed"), got), (waves, chans, occ)
    m.close()


@pytest.mark.parametrize("N", [7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 39, 40, 47, 48, 49,
                               55, 56, 62, 63, 64, 65, 71, 72, 73, 80, 87, 88, 95, 96])
def test_projected_region_counts(N):
    say(f"N={N}")
    _run(workload.make(N, FREQS, max(70, 32 * ((N + 31) // 32) + 1), 70, 7000 + N, batch="mixed",
                       rich=True), "projected")


@pytest.mark.parametrize("N,T", [(33, 1), (33, 7), (40, 8), (41, 9), (48, 16), (49, 17), (64, 24),
                                 (20, 25), (24, 31), (30, 32), (50, 33), (63, 40), (70, 41),
                                 (73, 57), (97, 63), (128, 20), (1, 66), (5, 70), (12, 30)])
def test_direct_bins(N, T):
    say(f"N={N} T={T}")
    _run(workload.make(N, FREQS, T, 70, 8000 + N + T, batch="mixed", rich=True), "direct",
         flags=lib().FGL_MIXED_DIRECT)


@pytest.mark.parametrize("na,nb,T", [(3, 5, 70), (2, 8, 70), (3, 8, 70), (5, 5, 70), (3, 11, 100),
                                     (3, 16, 100), (3, 17, 100), (4, 16, 100), (3, 21, 100),
                                     (2, 33, 130), (3, 24, 130), (5, 16, 130), (3, 32, 130),
                                     (3, 11, 20), (5, 13, 9), (7, 14, 33)])
def test_masks(na, nb, T):
    w = workload.make_masks(na, nb, FREQS, T, 70, 9000 + na * nb + T, batch="mixed")
    say(f"masks {na}x{nb} T={T}")
    _run(w, "projected" if T >= na * nb + 1 else "direct")
