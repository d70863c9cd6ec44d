"""Momentum in a uniform flow (GPU, FP64).  Without walls and forces the collision
leaves rho and j alone, and streaming changes nothing; what round-off does to
them must not build up.  200 steps of Q roundings of populations (2^-53 of a
value that is a tenth of j or less) that fall either way move j by a relative
sqrt(200 Q) 2^-53 / 10, at most 7e-16 in one flow and half of that as the root
mean square over many flows of any direction: 3.5e-16, the bound.  Round-off
that a collision repeats in every step gives three times as much."""

import numpy as np
import pytest

from gpu_util import require_gpu
from workloads import configs
from workloads import geometry as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("oblique", [False, True])
@pytest.mark.parametrize("lattice,shape", [("D2Q9", (16, 16, 1)), ("D3Q15", (8, 8, 8)), ("D3Q19", (8, 8, 8))])
def test_uniform_flow_keeps_its_momentum(lattice, shape, oblique):
    require_gpu()
    from paper_1712_08288_amd import binding
    rng = np.random.default_rng(3)
    e, _, _ = binding.lattice_info(lattice)
    e = e.astype(np.longdouble)
    geom = G.empty(lattice, shape)
    drift = []
    for _ in range(100):
        tau = rng.uniform(0.52, 1.2)
        rates = {"D2Q9": configs.d2q9_rates(tau), "D3Q15": configs.d3q15_paper_rates(1 / tau),
                 "D3Q19": configs.d3q19_rates(tau)}[lattice]
        u = np.zeros(e.shape[1])
        u[0] = rng.uniform(0.01, 0.08)
        if oblique:
            u[1:] = rng.uniform(-0.08, 0.08, size=u.size - 1)
        sv = binding.solver_for(geom, rates)
        sv.init(np.ones(geom.n_nodes), np.tile(u, (geom.n_nodes, 1)))
        j = []
        for n in (0, 200):
            sv.step(n)
            j.append(e.T @ sv.distribution()[:, 5].astype(np.longdouble))
        sv.close()
        drift.append(float(np.sqrt(((j[1] - j[0]) ** 2).sum() / (j[0] ** 2).sum())))
    assert np.sqrt(np.mean(np.square(drift))) < 3.5e-16
