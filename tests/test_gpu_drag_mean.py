"""The mean drag's round-off (GPU).  The momentum-exchange force holds the
constant 2 w_i rho0 e_ibar on every link, which cancels between the links of a
closed obstacle; its round-off must not stay behind in the mean.

The flow starts from deviations of 1e-6, so that the drag is about 1e-7 where
each link's constant is 0.1: the constant's round-off, kept in every link's sum
over 300 steps, is 1e-15 or a relative 1e-8, while the populations' own
round-off (1e-22 a step and link) and that of summing them (300 additions) is
below 1e-12 after a cancellation of 1e2 among the links.  The bound between the
two is 1e-10; an open wall, whose constant does not cancel, has 1e-13 of it."""

import math

import numpy as np
import pytest

from gpu_util import require_gpu
from workloads import configs, states
from workloads import geometry as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _mean_drag(o, df, steps, t0, t1, tag):
    """Exactly summed mean x force over steps t0 <= t < t1: (value, constant)."""
    ex = o.e[o.lk_dir, 0]
    on = (o.lk_tag == tag) & (ex != 0)
    dev = []

    def see(t, f, fp, fn):
        if t0 <= t < t1:
            for v in (fp[o.lk_opp, o.lk_node], fn[o.lk_dir, o.lk_node]):
                dev.append((-ex * v)[on])

    o.run(o.init_deviation(df), steps, see)
    const = math.fsum(np.concatenate([(-ex * 2 * o.w[o.lk_dir] * o.rho0)[on]]))
    return math.fsum(np.concatenate(dev)) / (t1 - t0) + const, const


CASES = {
    "cylinders": (lambda: G.random_cylinders(70, 45, 3, 4.0, 7.0, seed=31), 1, {}),
    "two_node": (lambda: G.random_cylinders(41, 33, 2, 4.0, 6.0, seed=8), 1, dict(two_node=True)),
    "open_wall": (lambda: G.channel_cylinder(60, 41, 5.2, (20.4, 20.3), 1e-6), 2, {}),
    "spheres": (lambda: G.random_spheres(30, 20, 18, 2, 3.0, 4.5, seed=2), 1, {}),
    "spheres_d3q15": (lambda: G.random_spheres(20, 18, 16, 2, 3.0, 4.5, seed=3, lattice="D3Q15"), 1, {}),
}


@pytest.mark.parametrize("single", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_mean_drag_keeps_no_round_off_of_the_constant(monkeypatch, name, single):
    from oracle.lbm import Oracle
    from paper_1712_08288_amd import binding
    make, tag, kw = CASES[name]
    geom = make()
    rates = {"D2Q9": configs.d2q9_rates(0.62), "D3Q15": configs.d3q15_paper_rates(1.2),
             "D3Q19": configs.d3q19_rates(0.7)}[geom.lattice]
    df = states.random_deviation(len(rates), geom.n_nodes, seed=3, amp=1e-6)
    if geom.x_bc == "outflow":
        from workloads.velocities import VELOCITIES
        df = states.outlet_consistent(df, geom.shape, VELOCITIES[geom.lattice])
    steps, t0, t1 = 321, 5, 305
    rho0 = 0.9
    want, const = _mean_drag(Oracle(geom, rates, rho0=rho0, l_rule="gamma2", **kw), df, steps, t0, t1, tag)
    if single:
        monkeypatch.setenv("LBM_DEBUG", "1")
    sv = binding.solver_for(geom, rates, rho0=rho0, l_rule="gamma2", **kw)
    sv.init_deviation(df)
    sv.set_objective("force_x", tag, t0, t1)
    for n in (7, 200, steps - 207):
        sv.step(n)
    got = sv.objective()
    sv.close()
    assert abs(got - want) < (1e-13 * abs(const) if name == "open_wall" else 1e-10 * abs(want)), (got, want)
