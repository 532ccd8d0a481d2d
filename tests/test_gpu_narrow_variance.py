"""Posterior variances in blocks of 1, 8, 16 and 32 right-hand sides: requests at
the edges of the widths, and one block's remainder after a full one, against
the oracle to 1e-8 of the prior (float64 matrix; the bound of the other variance
tests), with a site far from all data (its column is zero; the prior exactly)
and small and large preconditioner blocks (the LDS and the matrix-core update)."""
import numpy as np
import pytest

from gpu_util import dev, host
from oracle import predict
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cell", [0.03, 0.2])
@pytest.mark.parametrize("n", [3, 300, 800])
def test_widths(n, cell):
    import paper_2411_05869_amd as gp
    p = uniform_problem(n, 2, 90 + n, r0=0.12, n1=3, n2=2, bump_radius=0.25)
    ctx = gp.Context()
    K = ctx.assemble(ctx.dataset(dev(p.x), cell=np.full(2, cell)), p.theta, 0)
    rng = np.random.default_rng(n)
    xs = np.concatenate([np.full((1, 2), 9.0), rng.uniform(-0.1, 1.1, (41, 2))])
    ref, prior = predict.variance(xs, p.x, p.theta), predict.prior_variance(xs, p.theta)
    for precond in (gp.PRECOND_JACOBI, gp.PRECOND_BLOCK_JACOBI):
        for lo, m in ((0, 1), (1, 1), (0, 2), (1, 8), (0, 9), (1, 16), (0, 17), (1, 32), (0, 33), (1, 40), (0, 42)):
            v, r = ctx.predict_var(K, p.theta, dev(xs[lo:lo + m].copy()), precond=precond)
            v = host(v)
            assert r["status"] == 0 and r["relres"] <= 1e-10
            assert float(np.max(np.abs(v - ref[lo:lo + m]) / prior[lo:lo + m])) <= 1e-8, (lo, m)
            if lo == 0:
                assert v[0] == prior[0]
