"""The gradient over the lengths its staged quad rows can have (one to five
16-row tiles in FP32, the direct form; one to three in FP64, the projected one),
several stages of channels and quads that do not divide over the waves, against
the oracle's analytic gradient at the bar of tests/test_grad_gpu.py."""
import numpy as np
import pytest

import oracle
import workload
from tests.gpu_util import check, lib, say
from tests.test_grad_gpu import check_grad, term_scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,F,T,form", [
    (4, 151, 1, "direct"), (10, 37, 16, "direct"), (13, 18, 17, "direct"), (20, 17, 32, "direct"),
    (24, 17, 33, "direct"), (12, 9, 48, "direct"), (6, 9, 49, "direct"), (5, 7, 80, "direct"),
    (48, 6, 2, "direct"), (90, 3, 12, "direct"),
    (3, 33, 65, "projected"), (11, 18, 40, "projected"), (15, 17, 33, "projected"),
    (16, 17, 33, "projected"), (33, 5, 65, "projected"),
])
def test_gradient_over_row_lengths(N, F, T, form):
    fgl, orc = lib(), oracle.load()
    w = workload.make(N, np.linspace(50.0, 200.0, F), T, 19, 700 + N + T, batch="mixed")
    m = fgl.Model.from_workload(w, fgl.FGL_MIXED_DIRECT if form == "direct" else 0)
    say(f"gradient N={N} F={F} T={T} form={form}")
    if form == "projected":
        assert m.form in ("projected", "thin")       # thin models keep the projected gradient
    ll, g = m.loglike_grad(w.theta)
    rl, rg = orc.grad_w(w)
    check(ll, rl, "fp64", f"N{N}", theta=w.theta, n=w.F * w.T)
    check_grad(g, rg, term_scale(orc, w, w.theta), f"N{N}")
    m.close()
