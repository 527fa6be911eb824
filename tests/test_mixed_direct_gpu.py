"""The mixed kernel's direct form over its chunk counts, slot counts and mask kinds
(one to four chunks of regions; no masks, masks that fill half chunks and masks that
cross them), with one row tile and several, whole and ragged, against the FP64
oracle, and bit for bit between the tiles of a model."""
import numpy as np
import pytest

import oracle
import workload
from tests.gpu_util import check, lib, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nb", [(0, 20), (0, 40), (0, 64), (0, 70), (0, 96), (0, 97), (0, 128), (2, 16), (3, 16),
                                   (6, 16), (8, 16), (4, 32), (3, 10), (4, 10), (5, 12), (4, 17), (3, 30), (4, 30)])
def test_direct_form(na, nb):
    fgl, orc = lib(), oracle.load()
    N = max(na, 1) * nb
    for T in (1, 16, 31, 32, 33, 64, 71):
        freqs = np.linspace(50.0, 200.0, 9)
        w = (workload.make_masks(na, nb, freqs, T, 40, 800 + N + T, batch="mixed") if na else
             workload.make(nb, freqs, T, 40, 800 + N + T, batch="mixed"))
        m = fgl.Model.from_workload(w, fgl.FGL_MIXED_DIRECT)
        assert m.form == "direct"
        ref = orc.loglike_w(w)
        got = m.loglike(w.theta, "mixed")
        check(got, ref, "mixed", f"a{na} N{N} T{T}")
        n = 0
        for waves in (4, 8):
            for chans in range(1, 9):
                try:
                    m.set_tile(w.B, "mixed", waves, chans, 2)
                except fgl.FGLError:
                    continue
                assert np.array_equal(m.loglike(w.theta, "mixed"), got), (T, waves, chans)
                n += 1
        assert n
        m.close()
    say(f"  a{na} N{N}: {n} tiles")
