"""The link coefficients' rounding (GPU): made in double, operation by operation
as Eq. (213) and l(gamma) are written, whatever the device could fuse.  From
rest the first step leaves c4 3 w_i rho0 e_i.phi alone in every link's value,
bit for bit what the same operations give on the host."""

import numpy as np
import pytest

from gpu_util import require_gpu
from workloads import configs
from workloads import geometry as G
from workloads.velocities import VELOCITIES

pytestmark = pytest.mark.gpu

RULES = {"gamma": lambda g: g, "1.5gamma": lambda g: 1.5 * g, "2gamma": lambda g: 2.0 * g,
         "gamma2": lambda g: g * g, "gamma2+gamma": lambda g: g * g + g, "zero": lambda g: 0.0 * g,
         "min": lambda g: np.maximum(2.0 * g - 1.0, 0.0)}
WEIGHTS = {"D2Q9": {0: 4.0 / 9, 1: 1.0 / 9, 2: 1.0 / 36}, "D3Q15": {0: 2.0 / 9, 1: 1.0 / 9, 3: 1.0 / 72},
           "D3Q19": {0: 1.0 / 3, 1: 1.0 / 18, 2: 1.0 / 36}}


@pytest.mark.parametrize("rule", list(RULES))
@pytest.mark.parametrize("lattice", ["D2Q9", "D3Q15", "D3Q19"])
def test_wall_terms_are_rounded_as_written(lattice, rule):
    require_gpu()
    from paper_1712_08288_amd import binding
    geom = (G.random_cylinders(50, 37, 3, 3.0, 5.0, seed=21) if lattice == "D2Q9" else
            G.random_spheres(26, 19, 17, 2, 2.5, 4.0, seed=22, lattice=lattice))
    rng = np.random.default_rng(5)
    geom = geom.with_q((0.5 if rule == "zero" else 1.0) * (1.0 - rng.random(geom.n_links)))
    geom = geom.with_wall_u(0.01 * rng.normal(size=geom.wall_u.shape))
    rates = {"D2Q9": configs.d2q9_rates(0.62), "D3Q15": configs.d3q15_paper_rates(1.2),
             "D3Q19": configs.d3q19_rates(0.7)}[lattice]
    b, rho0 = 0.8, 0.9
    sv = binding.solver_for(geom, rates, rho0=rho0, l_rule=rule, b=b)
    sv.init_deviation(np.zeros((len(rates), geom.n_nodes)))
    sv.step(1)
    got = sv.distribution()[geom.dir, geom.node]
    sv.close()
    e = np.asarray(VELOCITIES[lattice], dtype=np.float64)[geom.dir]
    w = np.array([WEIGHTS[lattice][int(k)] for k in (e * e).sum(1)])
    phi = np.zeros(geom.n_links)
    for a in range(e.shape[1]):
        phi = phi + e[:, a] * geom.wall_u[:, a]
    den = 1.0 + RULES[rule](geom.q)
    assert np.array_equal(got, b * 2.0 / den * (3.0 * w * rho0 * phi))
