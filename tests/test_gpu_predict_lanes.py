"""The kriging mean's lane-group search at the edges of its parts: more
candidates than one list holds, more pencils than one round takes, request
sizes around the points of a block, and a context with an HBM budget (which
keeps no packed copy and no member lists).

Against the FP64 oracle, to the bounds of the other prediction tests: 1e-10
(FP64) and 2e-7 (mixed) of sum_q |C(x*, x_q)| |alpha_q|; every term is formed
as before and the sums differ only in order."""
import numpy as np
import pytest

from oracle import kernel, predict
from gpu_util import dev, host
from workloads import random_core, uniform_problem

pytestmark = pytest.mark.gpu

# (d, n, r0, cells per r0): dense windows (hundreds of candidates in a few
# pencils), many pencils (a fine grid), an almost empty set
SHAPES = [(1, 900, 0.3, 1.15), (2, 1200, 0.35, 1.15), (2, 700, 0.2, 0.07), (3, 900, 0.3, 0.21), (3, 5, 0.4, 1.15)]


@pytest.mark.parametrize("core", [0, 1, 2])
@pytest.mark.parametrize("d,n,r0,cell", SHAPES)
def test_lists_and_pencils(d, n, r0, cell, core):
    from paper_2411_05869_amd import Context
    p = uniform_problem(n, d, 7 * d + n, r0=r0, n1=3, n2=2, bump_radius=0.3)
    if core:
        p.theta.core = random_core(core, d, 3)
    rng = np.random.default_rng(n + d)
    alpha = rng.standard_normal(n)
    xs = rng.uniform(-0.1, 1.1, (67, d))
    xs[5] = np.nan
    xs[6] = 40.0
    ref = np.zeros(len(xs))
    ok = np.isfinite(xs).all(1)
    ref[ok] = predict.mean(xs[ok], p.x, p.theta, alpha)
    rp, cols, vals = kernel.cross_entries(xs[ok], p.x, p.theta)
    sc = np.full(len(xs), 1e-300)
    sc[ok] = [np.abs(vals[rp[i]:rp[i + 1]]) @ np.abs(alpha[cols[rp[i]:rp[i + 1]]]) + 1e-300
              for i in range(int(ok.sum()))]
    free, tight = Context(), Context()
    tight.set_hbm_budget(1 << 30)
    got = {}
    for name, ctx in (("free", free), ("tight", tight)):
        ds = ctx.dataset(dev(p.x), cell=np.full(d, r0 * cell))
        pred = ctx.predictor(ds, p.theta, dev(alpha))
        for prec, tol in ((0, 1e-10), (1, 2e-7)):
            m = host(ctx.predict(pred, dev(xs), precision=prec))
            assert m[5] == 0.0 and m[6] == 0.0
            err = float(np.max(np.abs(m - ref) / sc))
            assert err <= tol, (name, prec, err)
            got[name, prec] = m
            for k in (1, 15, 16, 17, 33):     # a row's value does not depend on its request
                assert np.array_equal(host(ctx.predict(pred, dev(xs[:k]), precision=prec)), m[:k], equal_nan=True)
    if core == 0:   # the same terms in the same order from either layout
        for prec in (0, 1):
            assert np.array_equal(got["free", prec], got["tight", prec])
