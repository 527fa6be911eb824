"""The projected gradient of 64 and 32 regions without masks, whose last row is
done in FP64 beside the tiles (as the entries between its row groups are), over
channel counts and batches that leave remainders, against the oracle's analytic
gradient.

The bar is that of tests/test_grad_gpu.py plus the rounding of the model values in
the projected sums.  A channel's projected residual e = z - R p is a sum of N + 1
products, so it is off by at most (N + 16) 2^-53 (|D| + sum_i |K_i| P_i) in the
2-norm (|.| over the channel's time bins, which the orthonormal basis keeps; N + 1
products and sums, under 15 roundings in a power, its exponent and the rows), and
the entry of region j, sum_f ln(nu) P_j R_j e / sigma^2, by that times
|ln nu| P_j |K_j| / sigma^2; once more for the oracle's own sums over time."""
import numpy as np
import pytest

import oracle
import workload
from tests.gpu_util import check, lib, say
from tests.test_grad_gpu import term_scale

pytestmark = pytest.mark.gpu


def rounding(w, theta):
    """Per row and spectral index, the bound above."""
    L = np.log(w.freqs / w.nu_ref)
    k = np.sqrt((w.K.astype(np.float64) ** 2).sum(2))          # [N, F]
    d = np.sqrt((w.data ** 2).sum(1))
    out = np.zeros(theta.shape)
    for b, th in enumerate(theta):
        p = np.exp(-np.outer(th[:w.N], L))                     # [N, F]
        off = (w.N + 16) * 2.0 ** -53 * (d + (k * p).sum(0))   # [F]
        out[b, :w.N] = 2 * (np.abs(L) * p * k * off).sum(1) / th[-1] ** 2
    return out


@pytest.mark.parametrize("more", [1, 33])
@pytest.mark.parametrize("N,F,B", [(64, 3, 8), (64, 5, 17), (64, 18, 33), (32, 3, 8), (32, 17, 70)])
def test_last_row_beside_the_tiles(N, F, B, more):
    fgl, orc = lib(), oracle.load()
    w = workload.make(N, np.linspace(50.0, 200.0, F), N + more, B, 600 + N, batch="mixed", rich=True)
    rl, rg = orc.grad_w(w)
    m = fgl.Model.from_workload(w)
    assert m.form == "projected"
    ll, g = m.loglike_grad(w.theta)
    check(ll, rl, "fp64", f"N{N}", theta=w.theta, n=w.F * w.T)
    ok = np.isfinite(rg).all(axis=1)
    assert ok.sum() >= B // 2 and np.all(np.isnan(g[~ok]))
    bar = 1e-9 * (np.abs(rg) + term_scale(orc, w, w.theta))[ok]
    own = rounding(w, w.theta)[ok]
    d = np.abs(g - rg)[ok]
    say(f"  N{N} F{F} T{N + more}: max|d|/bar={np.max(d / bar):.3f}, rounding up to {np.max(own / bar):.3f} of the bar, "
        f"max|d|/both={np.max(d / (bar + own)):.3f}")
    assert np.all(d <= bar + own)
    m.close()
