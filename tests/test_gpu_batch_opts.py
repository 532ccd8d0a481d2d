"""gp_loglik_batch refuses options out of range with GP_EINVAL, as the other
solving calls do, in its status and in every result's."""
import pytest

from gpu_util import dev
from workloads import uniform_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [dict(rtol=2.0), dict(max_iter=0), dict(n_probes=1), dict(n_lanczos=129),
                                 dict(precond=7), dict(solver=9)])
def test_options_out_of_range(bad):
    import paper_2411_05869_amd as gp
    p = uniform_problem(300, 2, 4, r0=0.1)
    ctx = gp.Context()
    K = ctx.assemble(ctx.dataset(dev(p.x), cell=p.cell), p.theta, 0)
    y = dev(p.z_std)
    with pytest.raises(gp.GPError) as e:
        ctx.loglik_batch([K, K], [y, y], **bad)
    assert e.value.status == 1  # GP_EINVAL
    r = ctx.loglik_batch([K, K], [y, y])  # and goes on working
    assert all(x["status"] == 0 for x in r)
