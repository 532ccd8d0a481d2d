"""Sites 10^9 cells and more outside the training box, with a radius that
reaches it all the same: every training point lies in the site's window.
Against the FP64 oracle, to the bound of the other prediction tests."""
import numpy as np
import pytest

from oracle import predict
from gpu_util import dev, host
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3])
def test_far_sites(d):
    import paper_2411_05869_amd as gp
    p = uniform_problem(60, d, 90 + d, r0=4e8, n1=1, n2=1, bump_radius=0.3)
    alpha = np.random.default_rng(d).random(p.n)  # one sign: no cancellation in the bound
    xs = np.full((4, d), 0.5)
    xs[0, 0], xs[1, 0], xs[2, 0], xs[3, 0] = -3e8, 3e8, -5e7, -3.99e8
    ctx = gp.Context()
    pred = ctx.predictor(ctx.dataset(dev(p.x), cell=np.full(d, 0.1)), p.theta, dev(alpha))
    ref = predict.mean(xs, p.x, p.theta, alpha)
    got = host(ctx.predict(pred, dev(xs)))
    assert np.all(ref > 0.0)
    assert np.all(np.abs(got - ref) <= 1e-10 * ref), (got, ref)
