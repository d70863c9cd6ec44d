"""A handle whose new geometry is refused late, after its tables were replaced
(GPU): nothing of the old geometry can be launched any more, and the next
geometry starts afresh."""

import numpy as np
import pytest

from gpu_util import require_gpu
from workloads import configs, states
from workloads import geometry as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# on tiles, and a domain that takes single steps
@pytest.mark.parametrize("make,rates", [
    (lambda: G.random_cylinders(70, 45, 3, 4.0, 7.0, seed=31), configs.d2q9_rates(0.62)),
    (lambda: G.random_spheres(48, 40, 36, 2, 3.0, 6.0, seed=22), configs.d3q19_rates(0.7))])
def test_refused_geometry_needs_a_new_one(make, rates):
    from paper_1712_08288_amd import binding
    geom = make()
    good = geom.with_q(np.full(geom.n_links, 0.4))
    bad = np.full(geom.n_links, 0.4)
    bad[geom.n_links // 2] = 0.75            # l = 0 is convex up to one half
    df = states.random_deviation(len(rates), geom.n_nodes, seed=3)
    sv = binding.solver_for(good, rates, l_rule="zero")
    sv.init_deviation(df)
    sv.set_objective("force_x", 1, 0, 5)
    sv.run_checkpointed(5, 2)
    sv.adjoint()
    want = [sv.distribution(), np.array(sv.objective()), sv.grad()["q"]]

    def refused(call):
        with pytest.raises(binding.LBMError) as ex:
            call()
        assert ex.value.name == "ESTATE"

    with pytest.raises(binding.LBMError) as ex:
        sv.set_geometry(geom.solid, geom.node, geom.dir, bad, geom.wall_u, geom.tag)
    assert ex.value.name == "EINVAL"
    for call in (lambda: sv.step(3), lambda: sv.moments(), lambda: sv.force(2), lambda: sv.reduce(),
                 lambda: sv.run_checkpointed(4, 2), lambda: sv.adjoint(), lambda: sv.grad(),
                 lambda: sv.init(), lambda: sv.update_links(good.q),
                 lambda: sv.set_objective("force_x", 1, 0, 5)):
        refused(call)
    sv.set_geometry(good.solid, good.node, good.dir, good.q, good.wall_u, good.tag)
    refused(lambda: sv.step(3))
    sv.init_deviation(df)
    sv.set_objective("force_x", 1, 0, 5)
    sv.run_checkpointed(5, 2)
    sv.adjoint()
    for a, b in zip([sv.distribution(), np.array(sv.objective()), sv.grad()["q"]], want):
        assert np.array_equal(a, b, equal_nan=True)
    sv.close()
