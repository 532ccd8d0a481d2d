"""The bump part of the kriging mean with a core kernel, over the groups' member
lists (from 4096 masked training points on, in a context without an HBM
budget) and over every masked point: points in one, several and no groups, on
both sides of that number.  Against the FP64 oracle, to the bounds of the other
prediction tests: 1e-10 (FP64) and 2e-7 (mixed) of sum_q |C(x*, x_q)| |alpha_q|."""
import numpy as np
import pytest

from oracle import kernel, predict
from gpu_util import dev, host
from workloads import random_core, uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("core", [1, 2])
@pytest.mark.parametrize("nm", [4095, 4096, 5121])
def test_lists(nm, core):
    from paper_2411_05869_amd import Context
    p = uniform_problem(6000, 2, 21, r0=0.03, n1=3, n2=1)
    # group 0: the nm points of smallest first coordinate; groups 1 and 2 inside it
    x0 = np.sort(p.x[:, 0])
    edge = 0.5 * (x0[nm - 1] + x0[nm])
    p.theta.h[:, 0] = (0.0, 0.5), (0.2, 0.3), (0.25, 0.5)
    p.theta.r[:, 0] = (edge, np.inf), (0.15, 0.2), (0.1, 0.3)
    p.theta.core = random_core(core, 2, 3)
    M, _ = kernel.features(p.x, p.theta)
    assert int(M.any(axis=1).sum()) == nm
    rng = np.random.default_rng(nm)
    alpha = rng.standard_normal(p.n)
    xs = rng.uniform(-0.1, 1.1, (150, 2))
    ref = predict.mean(xs, p.x, p.theta, alpha)
    rp, cols, vals = kernel.cross_entries(xs, p.x, p.theta)
    sc = np.array([np.abs(vals[rp[i]:rp[i + 1]]) @ np.abs(alpha[cols[rp[i]:rp[i + 1]]]) for i in range(len(xs))])
    for budget in (0, 1 << 30):
        ctx = Context()
        ctx.set_hbm_budget(budget)
        pred = ctx.predictor(ctx.dataset(dev(p.x), cell=p.cell), p.theta, dev(alpha))
        for prec, tol in ((0, 1e-10), (1, 2e-7)):
            got = host(ctx.predict(pred, dev(xs), precision=prec))
            assert np.all(np.abs(got - ref) <= tol * sc + 1e-300)
