"""Several steps per launch on tiles against one step per launch, bit for bit
(GPU).  LBM_DEBUG=1 steps one by one, so the two handles take the two paths;
the sizes are those at which a tile, its halo or the wrap inside a region
begins or ends, with every x boundary, both schemes, decaying wall data and a
drag window that opens and closes inside a launch."""

import numpy as np
import pytest

from gpu_util import require_gpu
from workloads import configs, states
from workloads import geometry as G
from workloads.velocities import VELOCITIES

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _seam(geom):
    geom.x_bc = "pressure"
    return geom


def _moving(geom, seed=1):
    return geom.with_wall_u(0.01 * np.random.default_rng(seed).normal(size=geom.wall_u.shape))


CASES = {
    # one region holds the whole period
    "all_wraps": (lambda: _moving(G.random_cylinders(20, 12, 1, 2.0, 2.9, seed=4)), {}),
    "one_column": (lambda: G.poiseuille_channel(9, 0.25, nx=1), dict(g=(1e-5, 0, 0))),
    # wraps in x only, tiles in y
    "narrow": (lambda: G.poiseuille_channel(81, 0.75, nx=2), dict(g=(1e-5, 0, 0), b=0.7)),
    "tiles": (lambda: _moving(G.random_cylinders(70, 45, 3, 4.0, 7.0, seed=31)), dict(decay=0.97)),
    "tiles_exact": (lambda: G.random_cylinders(64, 40, 2, 4.0, 7.0, seed=5), {}),
    "seam": (lambda: _seam(G.random_cylinders(131, 67, 5, 4.0, 7.0, seed=6)), dict(dp=1e-3)),
    "two_node": (lambda: _moving(G.random_cylinders(97, 61, 5, 4.0, 7.0, seed=7)),
                 dict(two_node=True, b=0.8)),
    "two_node_seam": (lambda: _seam(G.random_cylinders(33, 29, 2, 3.0, 5.0, seed=8)),
                      dict(two_node=True, dp=1e-3)),
    "outflow": (lambda: G.channel_cylinder(160, 71, 6.3, (30.4, 35.3), 0.03), {}),
    "outflow_wraps": (lambda: G.channel_cylinder(30, 19, 3.2, (12.4, 9.3), 0.03), {}),
    # more links in a region than threads of a block
    "dense": (lambda: G.random_cylinders(200, 190, 160, 2.0, 3.5, seed=9), {}),
    "pipe": (lambda: G.pipe(20.0, nx=2, lattice="D3Q15"), dict(g=(1e-6, 0, 0))),
    "pipe_d3q19": (lambda: G.pipe(7.0, nx=2, lattice="D3Q19"), dict(g=(1e-6, 0, 0), two_node=True)),
    "pipe_seam": (lambda: _seam(G.pipe(9.0, nx=3, lattice="D3Q19")), dict(dp=1e-4)),
}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_tiles_equal_single_steps(monkeypatch, name, precision):
    import torch
    from paper_1712_08288_amd import binding
    make, kw = CASES[name]
    geom = make()
    rates = {"D2Q9": configs.d2q9_rates(0.62), "D3Q15": configs.d3q15_paper_rates(1.2),
             "D3Q19": configs.d3q19_rates(0.7)}[geom.lattice]
    df = states.random_deviation(len(rates), geom.n_nodes, seed=3)
    if geom.x_bc == "outflow":
        df = states.outlet_consistent(df, geom.shape, VELOCITIES[geom.lattice])
    tag = int(geom.tag.max())
    out = {}
    for mode in ("0", "1"):
        monkeypatch.setenv("LBM_DEBUG", mode)
        sv = binding.solver_for(geom, rates, g=kw.get("g"), dp=kw.get("dp", 0.0), l_rule="gamma2",
                                b=kw.get("b", 1.0), two_node=kw.get("two_node", False),
                                precision=precision)
        sv.set_wall_decay(kw.get("decay", 1.0))
        sv.init_deviation(df)
        got = []
        for n in (1, 2, 7, 33):
            sv.set_objective("force_x", tag, sv.time + 1, sv.time + n + 1)
            sv.step(n)
            got += [sv.distribution(), np.array(sv.objective()), sv.force(tag + 1)]
        # drag only within a window of the steps, then the gradient
        sv.set_objective("force_x", tag, sv.time + 3, sv.time + 14)
        sv.run_checkpointed(17, 6)
        sv.adjoint()
        gr = sv.grad()
        got += [np.array(sv.objective()), sv.distribution()] + [gr[k] for k in ("q", "wall_u", "g", "s")]
        state = torch.empty(sv.state_bytes(), dtype=torch.uint8, device="cuda")
        sv.get_state(state)
        out[mode] = got
        assert np.all(np.isfinite(got[-2])) and sv.time == 60
        sv.close()
    for k, (a, b) in enumerate(zip(out["0"], out["1"])):
        assert np.array_equal(a, b, equal_nan=True), k
