"""Products written in the caller's order by the last pass over each row: with
and without group rows, rows of more than 128 entries, one to 32 columns,
FP64 and mixed, small and above the one-launch product's limits, into an output
that also is the input (the C ABI allows it: x is read before y is written).

A product's columns are the matrix's own columns scaled: K e_j is checked
against the exported matrix (bitwise where a row's sum has one term)."""
import ctypes as C

import numpy as np
import pytest

from gpu_util import dev, export, host, to_scipy
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,r0,n1", [(1, 0.1, 1), (600, 0.05, 3), (900, 0.35, 3), (500, 0.2, 0)])
def test_columns_of_the_matrix(n, r0, n1, prec):
    import torch
    import paper_2411_05869_amd as gp
    p = uniform_problem(n, 2, 30 + n, r0=r0, n1=n1, n2=2 if n1 else 0, bump_radius=0.3)
    ctx = gp.Context()
    K = ctx.assemble(ctx.dataset(dev(p.x), cell=p.cell), p.theta, prec)
    A = to_scipy(*export(ctx, K), n).toarray()
    rng = np.random.default_rng(n)
    for k in (1, 2, 5, 16, 20, 32):
        j = rng.integers(0, n, k)
        X = np.zeros((n, k))
        X[j, np.arange(k)] = 1.0
        x = dev(X if k > 1 else X[:, 0])
        Y = host(ctx.matvec(K, x)).reshape(n, k)
        assert np.array_equal(Y, A[:, j]), k
        # in place
        ctx._check(ctx._L.gp_matvec(ctx._h, K._h, k, C.c_void_p(x.data_ptr()), C.c_void_p(x.data_ptr())), "gp_matvec")
        assert np.array_equal(host(x).reshape(n, k), A[:, j]), k
    x = dev(rng.standard_normal(n))
    assert torch.equal(ctx.matvec_noalloc(K, x, torch.empty_like(x)), ctx.matvec(K, x))
