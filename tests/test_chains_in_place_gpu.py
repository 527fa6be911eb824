"""Chains whose rounds run inside one workgroup (small models) against the
launched rounds, bit for bit.

Kernel timing keeps a call on the launched rounds, so the same engine seed
gives the same chains both ways.  The cases cover every compiled region count,
channel counts around the group and wave sizes, several channel passes per
round, amplitude masks, models without the 21-cm term, zero steps, rows outside
the box and a call longer than one launch.
"""
import numpy as np
import pytest

import workload
from paper_2603_13196_amd import sampler as ns
from tests.gpu_util import lib, say

pytestmark = pytest.mark.gpu


def _both(fgl, model, lo, hi, n, steps, prec, calls=2, spread=0.05, quantile=0.2, scale=None):
    rng = np.random.Generator(np.random.PCG64(n * 1000 + steps))
    mid = (lo + hi) / 2
    z = np.clip(mid + spread * (hi - lo) * rng.standard_normal((5 * n, lo.size)), lo, hi)
    lz = model.loglike(ns.to_theta(z), prec)
    lstar = float(np.quantile(lz, quantile)) if quantile is not None else -np.inf
    order = np.argsort(lz)[-n:]
    chol = np.linalg.cholesky(np.cov(z.T) + 1e-9 * np.eye(lo.size))
    if scale is not None:
        chol = chol * scale
    got = []
    for timed in (False, True):
        eng = fgl.Chains(model, n, lo, hi, seed=77)
        model.kernel_timing(timed)
        got.append([eng.run(z[order], lz[order], lstar, chol, steps, prec) for _ in range(calls)])
        model.kernel_timing(False)
        eng.close()
    for a, b in zip(*got):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        assert a[2:] == b[2:]
    say(f"  n={n} steps={steps}: evals {got[0][0][2]} rounds {got[0][0][3]}")


@pytest.mark.parametrize("N,F,T,n,steps", [
    (1, 1, 1, 3, 5), (3, 11, 4, 64, 8), (4, 64, 64, 17, 4), (7, 65, 40, 9, 4), (10, 151, 1, 70, 12),
    (12, 151, 20, 31, 3), (16, 301, 20, 20, 3), (24, 127, 9, 16, 3), (32, 190, 8, 16, 3),
    (8, 701, 2, 12, 4),
])
def test_in_place_chains_equal_launched_chains(N, F, T, n, steps):
    fgl = lib()
    w = workload.make(N, np.linspace(50.0, 200.0, F), T, 8, 4000 + N + T)
    model = fgl.Model.from_workload(w)
    assert model.form == "thin"
    lo, hi = ns.foreground_box(N)
    _both(fgl, model, lo, hi, n, steps, "mixed" if N % 2 else "fp64")
    model.close()


def test_in_place_chains_with_masks_and_without_21cm():
    fgl = lib()
    w = workload.make_masks(3, 4, np.linspace(50.0, 200.0, 40), 5, 8, 91)
    model = fgl.Model.from_workload(w)
    lo, hi = ns.foreground_box(4, n_alpha=3)
    _both(fgl, model, lo, hi, 33, 5, "mixed")
    model.close()
    w = workload.make(5, np.linspace(50.0, 200.0, 40), 3, 8, 92)
    model = fgl.Model.from_workload(w, flags=fgl.FGL_NO_21CM)
    lo, hi = ns.foreground_box(5, no21=True)
    _both(fgl, model, lo, hi, 33, 5, "mixed")
    model.close()


def test_in_place_chains_at_the_edges():
    """No steps; steps far wider than the box, so that most proposals are
    outside it; a flat constraint; and more rounds than one launch takes."""
    fgl = lib()
    w = workload.make(3, np.linspace(60.0, 190.0, 11), 2, 8, 93)
    model = fgl.Model.from_workload(w)
    lo, hi = ns.foreground_box(3)
    _both(fgl, model, lo, hi, 10, 0, "mixed")
    _both(fgl, model, lo, hi, 40, 6, "mixed", scale=200.0)
    _both(fgl, model, lo, hi, 10, 6, "mixed", quantile=None, scale=1e-3)
    _both(fgl, model, lo, hi, 4, 700, "mixed", calls=1)
    model.close()
