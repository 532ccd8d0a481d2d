"""The SLQ quadrature (trapezoidal rule for e_1^T log(T) e_1) against the
oracle's eigenvalue quadrature with identical probes, at the step counts where
its parts change (one step, the first division, a wave's width, the maximum)
and probe counts around the probes of a block and a block of 32.

Both sides re-orthogonalise, so their coefficients agree to rounding; each
probe's n e_1^T log(T) e_1 then carries an error of a few hundred eps times n
on either side (cond T < 1e4 here), and 1e-10 n bounds their difference."""
import pytest

from gpu_util import dev, host  # noqa: F401
from oracle import kernel, slq
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [1, 2, 3, 63, 64, 65, 127, 128])
@pytest.mark.parametrize("probes", [2, 5, 33])
def test_quadrature_matches_eigenvalues(steps, probes):
    import scipy.sparse as sp
    from paper_2411_05869_amd import LOGDET_SLQ_REORTH, Context
    p = uniform_problem(400, 2, 17, r0=0.09, n1=2, n2=2, bump_radius=0.2)
    K, _ = kernel.dense(p.x, p.theta)
    ref = slq.slq_logdet(sp.csr_matrix(K), seed=11, n_probes=probes, n_steps=steps, reorth=True)
    ctx = Context()
    Kg = ctx.assemble(ctx.dataset(dev(p.x), cell=p.cell), p.theta, 0)
    r = ctx.loglik(Kg, dev(p.z_std), seed=11, n_probes=probes, n_lanczos=steps, logdet_mode=LOGDET_SLQ_REORTH)
    assert r["lanczos_steps"] == int(max(ref["steps"]))
    assert abs(r["logdet"] - ref["logdet"]) <= 1e-10 * p.n
    assert abs(r["logdet_se"] - ref["se"]) <= 1e-10 * p.n
