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
    # well conditioned: eight iterations take the recursion below a bound that rounding keeps the
    # recomputed residual above
    p = uniform_problem(1500, 2, 78, r0=0.02, n1=0, n2=0, nugget=1.0)
    ctx = gp.Context()
    K = ctx.assemble(ctx.dataset(dev(p.x), cell=p.cell), p.theta, 0)
    y, a = dev(p.z_std), torch.empty(p.n, dtype=torch.float64, device="cuda")

    def solve():
        return ctx.solve(K, y, a, rtol=1e-17, max_iter=24, solver=gp.SOLVER_CG, raise_on_error=False)

    for _ in range(100):
        r = solve()
    assert r["cg_iters"] == 24 and r["refreshes"] == 3  # refused after each of its blocks, the first among them
    before = _host_bytes()
    solves = 200
    for _ in range(solves):
        solve()
    grown = (_host_bytes() - before) / solves
    assert grown <= 33 * 300 / 2, f"{grown:.0f} bytes a solve"
