"""The block-Jacobi products at the edges of their parts: blocks of one row, of
a few, of exactly 32 and of cells split at 32 points, row counts around a tile
of 64 rows and a step's 512, mean blocks on either side of the matrix-core
rule (variance) and of the step's prefetch rule (solve).

The solution does not depend on the preconditioner, so both solves are held to
the oracle: variances to 1e-8 of the prior, as the other variance tests;
weights at rtol 1e-12 to 1e-8 relative (the residual bound times cond K < 1e4)."""
import numpy as np
import pytest

from gpu_util import dev, host
from oracle import kernel, likelihood, predict
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 33, 63, 64, 65, 128, 511, 513, 700])
@pytest.mark.parametrize("cell", [0.02, 0.12, 0.25, 3.0])
def test_block_sizes(n, cell):
    import torch
    from paper_2411_05869_amd import PRECOND_BLOCK_JACOBI, Context
    p = uniform_problem(n, 2, 40 + n, r0=0.15, n1=2, n2=2, bump_radius=0.3)
    K, _ = kernel.dense(p.x, p.theta)
    y = p.z_std
    ref = likelihood.dense_cholesky(K, y)
    ctx = Context()
    ds = ctx.dataset(dev(p.x), cell=np.full(2, cell))
    Kg = ctx.assemble(ds, p.theta, 0)
    alpha = torch.empty(n, dtype=torch.float64, device="cuda")
    r = ctx.solve(Kg, dev(y), alpha, rtol=1e-12, precond=PRECOND_BLOCK_JACOBI)
    assert r["status"] == 0
    assert np.linalg.norm(host(alpha) - ref["alpha"]) <= 1e-8 * np.linalg.norm(ref["alpha"])
    assert abs(r["quad"] - ref["quad"]) <= 1e-9 * abs(ref["quad"])
    xs = np.random.default_rng(n).uniform(-0.1, 1.1, (33, 2))
    v, rv = ctx.predict_var(Kg, p.theta, dev(xs), precond=PRECOND_BLOCK_JACOBI)
    prior = predict.prior_variance(xs, p.theta)
    assert rv["status"] == 0
    assert float(np.max(np.abs(host(v) - predict.variance(xs, p.x, p.theta)) / prior)) <= 1e-8
