"""Products with 2 .. 31 columns against the oracle's matrix, at the edges of the
column widths (2, 4, 8, 16, 32), with rows of more than 128 entries (a block
each), rows with and without a group part, fewer rows than a block takes, and
with the column ids as int32 (first) and as int16 offsets (once a one-column
product has built them).  Bounds as the other products: the sum's order is the
only difference, 1e-13 |K| |x| (and float32 values, 2^-24, in the mixed form)."""
import numpy as np
import pytest

from gpu_util import dev, host
from oracle import kernel
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,r0", [(1, 0.1), (15, 0.2), (17, 0.9), (700, 0.05), (900, 0.4)])
def test_narrow_products(n, r0, prec):
    import paper_2411_05869_amd as gp
    p = uniform_problem(n, 2, 60 + n, r0=r0, n1=3, n2=2, bump_radius=0.3)
    A = kernel.to_scipy(*kernel.sparse(p.x, p.theta), p.n)
    tol = 1e-13 if prec == 0 else 2.0 ** -24 + 1e-13
    ctx = gp.Context()
    K = ctx.assemble(ctx.dataset(dev(p.x), cell=p.cell), p.theta, prec)
    rng = np.random.default_rng(n)
    for offsets in (False, True):
        if offsets:
            ctx.matvec(K, dev(rng.standard_normal(n)))
        for k in (2, 3, 4, 5, 8, 9, 15, 16, 17, 31):
            X = rng.standard_normal((n, k))
            Y = host(ctx.matvec(K, dev(X)))
            bound = abs(A) @ np.abs(X)
            assert np.all(np.abs(Y - A @ X) <= tol * bound + 1e-300), (offsets, k)
