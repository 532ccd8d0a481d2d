"""A solve records its block of iterations at most once and gives it back: a
solve whose first block looks converged and is refused by the recomputed residual
comes past the point of recording a second time.

A lost executable graph keeps its 33 kernel nodes, each with a copy of its
arguments (100 bytes at least) and a node object of several times that: more
than 33 x 300 bytes, of which half is allowed here per solve."""
import ctypes as C

import pytest

from gpu_util import dev
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


class _Mallinfo2(C.Structure):
    _fields_ = [(f, C.c_size_t) for f in ("arena", "ordblks", "smblks", "hblks", "hblkhd", "usmblks", "fsmblks",
                                          "uordblks", "fordblks", "keepcost")]


def _host_bytes():
    f = C.CDLL(None).mallinfo2
    f.restype = _Mallinfo2
    i = f()
    return i.uordblks + i.hblkhd


def test_refused_convergence_leaves_nothing():
    import torch
    import paper_2411_05869_amd as gp
    # a nugget of 100 times the variance: eight iterations take the recursion to 1e-18 |y|, while
    # rounding keeps the recomputed residual above 1e-16 |y|
    p = uniform_problem(1500, 2, 78, r0=0.02, n1=0, n2=0, nugget=100.0)
    ctx = gp.Context()
    K = ctx.assemble(ctx.dataset(dev(p.x), cell=p.cell), p.theta, 0)
    y, a = dev(p.z_std), torch.empty(p.n, dtype=torch.float64, device="cuda")

    def solve(max_iter=24):
        return ctx.solve(K, y, a, rtol=1e-17, max_iter=max_iter, solver=gp.SOLVER_CG, precond=gp.PRECOND_JACOBI,
                         raise_on_error=False)

    assert solve(8)["refreshes"] == 1  # the first block looks converged
    for _ in range(100):
        r = solve()
    assert r["cg_iters"] == 24 and r["refreshes"] >= 1  # and is refused
    before = _host_bytes()
    solves = 200
    for _ in range(solves):
        solve()
    grown = (_host_bytes() - before) / solves
    assert grown <= 33 * 300 / 2, f"{grown:.0f} bytes a solve"
