"""Calls whose lanes exceed one launch (2^32 threads): the rows are taken in
ranges, with the values of small calls."""
import numpy as np
import pytest

from gpu_util import dev
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


def test_predict_of_more_rows_than_a_launch_takes():
    """Sixteen lanes a site: 2^28 sites are 2^32 threads.  The sites repeat a
    short request, so every row has to hold that request's value, bitwise; in the
    batch the last request's predictor starts inside a range."""
    import torch
    import paper_2411_05869_amd as gp
    m, period = (1 << 28) + 5, 1 << 18
    p = uniform_problem(40, 1, 5, r0=0.1, n1=1, n2=1, bump_radius=0.3)
    ctx = gp.Context()
    ds = ctx.dataset(dev(p.x), cell=p.cell)
    preds = [ctx.predictor(ds, p.theta, dev(s * p.z_std)) for s in (1.0, -2.0)]
    base = dev(np.random.default_rng(1).random((period, 1)))
    short = [ctx.predict(q, base) for q in preds]
    xs = torch.empty((m, 1), dtype=torch.float64, device="cuda")
    whole = m // period
    xs[:whole * period].view(whole, period).copy_(base.view(1, period).expand(whole, period))
    xs[whole * period:] = base[:m - whole * period]

    def rows_equal(out, ref, lo, hi):  # rows lo .. hi - 1 of the tiled request
        a, b = -(-lo // period), hi // period
        return (bool((out[a * period:b * period].view(b - a, period) == ref).all())
                and torch.equal(out[lo:a * period], ref[period - (a * period - lo):])
                and torch.equal(out[b * period:hi], ref[:hi - b * period]))

    out = ctx.predict(preds[0], xs)
    assert rows_equal(out, short[0], 0, m)
    cut = (1 << 27) + 9
    out = ctx.predict_batch([preds[0], preds[0], preds[1]], xs, [0, cut, cut, m], out=out.fill_(np.nan))
    assert rows_equal(out, short[0], 0, cut) and rows_equal(out, short[1], cut, m)


def test_narrow_product_of_more_rows_than_a_launch_takes():
    """Sixty-four lanes a row for 17 columns: 2^26 rows are 2^32 threads.  The
    points are further apart than the radius, so row p of the product is its
    diagonal value times x_p: one term, exact."""
    import torch
    import paper_2411_05869_amd as gp
    n, k = (1 << 26) + 3, 17
    p = uniform_problem(8, 1, 5, r0=0.5, n1=0, n2=0, nugget=0.25)
    ctx = gp.Context()
    x = torch.arange(n, dtype=torch.float64, device="cuda").view(n, 1)
    K = ctx.assemble(ctx.dataset(x, cell=[8.0]), p.theta, gp.MIXED)
    assert K.nnz == n
    X = torch.rand((n, k), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    Y = ctx.matvec(K, X)
    assert torch.equal(Y, X.mul_(1.25))
