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


# one bump over 96% of the points: 74.6M entries in group rows (two launches, 64M
# at most in one), and 8.3M (one launch, float32 values held to six waves from 4M)
@pytest.mark.parametrize("n,prec", [(9000, 0), (9000, 1), (3000, 1)])
def test_large_products_with_groups(n, prec):
    import torch
    import paper_2411_05869_amd as gp
    from oracle import kernel
    p = uniform_problem(n, 2, 30, r0=0.05, n1=1, n2=1)
    p.theta.h[0, 0, 0], p.theta.r[0, 0] = 0.5, (0.48, np.inf)
    ctx = gp.Context()
    K = ctx.assemble(ctx.dataset(dev(p.x), cell=p.cell), p.theta, prec)
    assert (K.nnz > 64 << 20) if n == 9000 else (4 << 20 < K.nnz < 64 << 20)
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n)
    y = ctx.matvec(K, dev(x))
    assert torch.equal(ctx.matvec_noalloc(K, dev(x), torch.empty_like(y)), y)
    M, F = kernel.features(p.x, p.theta)
    inside = M.any(axis=1)
    # rows with a group part, rows with one and local entries outside the group, rows without
    edge = np.nonzero(inside & (np.abs(p.x[:, 0] - 0.5) > 0.46))[0]
    rows = np.concatenate([rng.choice(np.nonzero(inside)[0], 20, replace=False), edge[:20],
                           rng.choice(np.nonzero(~inside)[0], 20, replace=False)])
    tol = 1e-13 if prec == 0 else 2.0 ** -24 + 1e-13
    got = host(y)
    for r in rows:
        c, v = kernel.row(p.x, p.theta, int(r), M, F)
        assert abs(got[r] - v @ x[c]) <= tol * (np.abs(v) @ np.abs(x[c])), r
