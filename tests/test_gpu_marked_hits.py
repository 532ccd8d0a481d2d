"""The fill that marks a scan's hits before it forms their entries (one row per
lane: more than 262,144 rows, 131,072 in three dimensions), with scans of fewer
and of more than 32 candidates and a cluster of more points than a wave stages,
for every core kind it serves: pattern bit-exact with the oracle, values to
1e-12, bitwise symmetric, as in the other assembly tests."""
import numpy as np
import pytest

from test_gpu_split_rows import _check
from workloads import random_core, uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,r0,core", [(1, 262150, 4e-5, 0), (2, 262145, 2e-3, 0), (2, 262145, 1.5e-3, 1),
                                         (3, 131073, 0.02, 1), (3, 131075, 0.015, 2)])
def test_marked_hits(d, n, r0, core):
    p = uniform_problem(n, d, 15 + d, r0=r0, n1=2, n2=1, bump_radius=min(0.02, 8 * r0))
    rng = np.random.default_rng(n)
    p.x[:400] = 0.37 + 0.3 * r0 * rng.standard_normal((400, d))
    if core:
        p.theta.core = random_core(core, d, 2)
    _check(p, core % 2, p.cell)
