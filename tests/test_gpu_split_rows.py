"""The local passes of the assembly on both sides of their rules: rows split
over eight lanes (count up to 131,072 rows, 65,536 in three dimensions; fill
up to twice that) and one row per lane beyond, with windows of fewer and of
many more candidates than a group of lanes takes, an empty neighbourhood, rows
with a bump group and every core kind.

Pattern bit-exact with the oracle, values to 1e-12 (float64) and one float32
rounding (mixed), bitwise symmetric, as in the other assembly tests."""
import numpy as np
import pytest

from gpu_util import assert_pattern_equal, dev, export, to_scipy, value_errors
from oracle import kernel
from workloads import random_core, uniform_problem

pytestmark = pytest.mark.gpu


def _check(p, prec, cell):
    from paper_2411_05869_amd import Context
    ctx = Context()
    K = ctx.assemble(ctx.dataset(dev(p.x), cell=cell), p.theta, prec)
    rp, col, val = export(ctx, K)
    ip, ci, vo = kernel.sparse(p.x, p.theta)
    assert_pattern_equal(rp, col, ip, ci)
    assert value_errors(val, vo) <= (1e-12 if prec == 0 else 1.2e-7)
    A = to_scipy(rp, col, val, p.n)
    assert (A != A.T).nnz == 0


@pytest.mark.parametrize("d,n,r0", [(1, 131072, 2e-5), (1, 262145, 1e-5), (2, 131073, 2e-3), (2, 262144, 1.5e-3),
                                    (2, 262145, 1.5e-3), (3, 65536, 0.02), (3, 65537, 0.02), (3, 131073, 0.015)])
def test_both_sides_of_the_rules(d, n, r0):
    p = uniform_problem(n, d, 5 + d, r0=r0, n1=2, n2=1, bump_radius=min(0.02, 8 * r0))
    _check(p, n % 2, p.cell)


@pytest.mark.parametrize("core", [0, 1, 2])
@pytest.mark.parametrize("d,n,r0,cell", [(1, 1, 0.1, 1.15), (1, 300, 0.4, 1.15), (2, 9, 0.01, 1.15), (2, 500, 0.3, 0.3),
                                         (2, 700, 0.3, 3.0), (3, 400, 0.35, 0.4), (3, 17, 0.9, 1.15)])
def test_window_sizes(d, n, r0, cell, core):
    p = uniform_problem(n, d, 60 + n, r0=r0, n1=2, n2=2, bump_radius=0.2)
    if core:
        p.theta.core = random_core(core, d, 2)
    for prec in (0, 1):
        _check(p, prec, np.full(d, r0 * cell))


# pencils of 9 to 10 candidates: the limits themselves and one row past them
@pytest.mark.parametrize("d,n,r0", [(2, 131072, 4.3e-3), (2, 131073, 4.3e-3), (2, 262144, 3e-3), (2, 262145, 3e-3),
                                    (3, 65536, 0.032), (3, 65537, 0.032), (3, 131072, 0.0253)])
def test_long_pencils_at_the_limits(d, n, r0):
    p = uniform_problem(n, d, 5 + d, r0=r0, n1=2, n2=1, bump_radius=2 * r0)
    _check(p, n % 2, p.cell)
