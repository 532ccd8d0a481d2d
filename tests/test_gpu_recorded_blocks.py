"""The recorded blocks of iterations of the conjugate gradients: the same bits
as plain launches (a context with its profile on launches plainly), whatever
the iteration count is against the block of eight, and a solve that goes on
after a recomputed residual (rtol below what the recursion keeps)."""
import pytest

from gpu_util import dev
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_iter", [7, 8, 9, 15, 16, 17, 24, 25, 31, 40, 2000])
@pytest.mark.parametrize("block", [False, True])
@pytest.mark.parametrize("rtol", [1e-10, 3e-16])
def test_recorded_blocks(max_iter, block, rtol):
    import torch
    import paper_2411_05869_amd as gp
    p = uniform_problem(1500, 2, 77, r0=0.1, n1=3, n2=2, bump_radius=0.25)
    y = dev(p.z_std)
    if rtol < 1e-12:
        max_iter = min(max_iter, 200)
    out = []
    for plain in (True, False):
        ctx = gp.Context()
        if plain:
            ctx.profile(True)
        K = ctx.assemble(ctx.dataset(dev(p.x), cell=p.cell), p.theta, 0)
        opts = dict(rtol=rtol, max_iter=max_iter,
                    precond=gp.PRECOND_BLOCK_JACOBI if block else gp.PRECOND_JACOBI, raise_on_error=False)
        runs = []
        for _ in range(2):  # a second solve records anew
            a = torch.empty(p.n, dtype=torch.float64, device="cuda")
            r = ctx.solve(K, y, a, **opts)
            b = torch.empty_like(a)
            rl = ctx.loglik(K, y, alpha_out=b, n_lanczos=10, **opts)  # the log det beside it
            runs.append((r, rl))
            assert torch.equal(a, b)
        out.append((a, [{k: v for k, v in r.items() if not k.startswith("t_")} for rr in runs for r in rr]))
    assert torch.equal(out[0][0], out[1][0])
    for r0, r1 in zip(out[0][1], out[1][1]):
        for k in ("status", "cg_iters", "relres", "quad", "logdet"):
            assert r0[k] == r1[k] or (r0[k] != r0[k] and r1[k] != r1[k]), k
