"""Replacing the link data (GPU): from host arrays and from device tensors, in
a caller's order that is not sorted, against a handle whose geometry was set
with those data and against the oracle; refused values change nothing."""

import numpy as np
import pytest

from gpu_util import rel_l2, require_gpu
from workloads import configs, states
from workloads import geometry as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _geometry(lattice, seed=3):
    if lattice == "D2Q9":
        geom = G.random_cylinders(50, 37, 3, 3.0, 5.0, seed=21)
    else:
        geom = G.random_spheres(26, 19, 17, 2, 2.5, 4.0, seed=22, lattice=lattice)
    o = np.random.default_rng(seed).permutation(geom.n_links)
    return G.Geometry(lattice, geom.shape, geom.solid, geom.node[o], geom.dir[o], geom.q[o],
                      geom.wall_u[o], geom.tag[o], geom.x_bc, dict(geom.meta))


RATES = {"D2Q9": configs.d2q9_rates(0.62), "D3Q15": configs.d3q15_paper_rates(1.2),
         "D3Q19": configs.d3q19_rates(0.7)}


def _run(sv, df, steps=9):
    sv.init_deviation(df)
    sv.set_objective("force_x", 1, 0, steps)
    sv.run_checkpointed(steps, 3)
    sv.adjoint()
    gr = sv.grad()
    return [sv.distribution()] + [gr[k] for k in ("q", "wall_u", "g", "s")]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("two_node", [False, True])
@pytest.mark.parametrize("lattice,rule", [("D2Q9", "gamma"), ("D2Q9", "min"), ("D2Q9", "zero"),
                                          ("D3Q15", "gamma2+gamma"), ("D3Q15", "1.5gamma"),
                                          ("D3Q19", "gamma2"), ("D3Q19", "2gamma")])
def test_update_equals_a_new_geometry(lattice, rule, two_node, precision):
    import torch
    from paper_1712_08288_amd import binding
    from oracle.lbm import Oracle
    geom = _geometry(lattice)
    rng = np.random.default_rng(5)
    top = 0.5 if rule == "zero" else 1.0     # l = 0 is convex up to one half
    q0 = np.minimum(geom.q, top)
    q = top * (1.0 - rng.random(geom.n_links))
    q[:3] = (top, 1e-9, 0.5)
    wu = 0.01 * rng.normal(size=geom.wall_u.shape)
    df = states.random_deviation(len(RATES[lattice]), geom.n_nodes, seed=3)
    kw = dict(precision=precision, l_rule=rule, b=0.8, two_node=two_node)
    sv = binding.solver_for(geom.with_q(q).with_wall_u(wu), RATES[lattice], **kw)
    want = _run(sv, df)
    sv.close()
    sv = binding.solver_for(geom.with_q(q0), RATES[lattice], **kw)
    for host in (True, False):
        sv.update_links(q0, np.zeros_like(wu))
        if host:
            sv.update_links(q)                # the other keeps its values
            sv.update_links(wall_u=wu)
        else:
            sv.update_links(torch.tensor(q, device="cuda"), torch.tensor(wu, device="cuda"))
        for a, b in zip(_run(sv, df), want):
            assert np.array_equal(a, b, equal_nan=True)
    # refused: nothing changes
    bad = [np.where(np.arange(len(q)) == 7, v, q) for v in (0.0, -0.1, np.nan, 1.0 + 1e-9)]
    if rule == "zero":
        bad.append(np.where(np.arange(len(q)) == 7, 0.6, q))
    for v in bad:
        for x in (v, torch.tensor(v, device="cuda")):
            with pytest.raises(binding.LBMError) as ex:
                sv.update_links(x, 0 * wu)
            assert ex.value.name == "EINVAL"
            if rule == "zero" and v[7] == 0.6:
                assert "at link 7 " in str(ex.value)
    for a, b in zip(_run(sv, df), want):
        assert np.array_equal(a, b, equal_nan=True)
    with pytest.raises(ValueError):
        sv.update_links(torch.zeros(3, dtype=torch.float64, device="cuda"))
    sv.close()
    o = Oracle(geom, RATES[lattice], l_rule=rule, b=0.8, q=q, wall_u=wu, two_node=two_node,
               allow_nonconvex=True)
    f = o.run(o.init_deviation(df), 9)
    # the forward tests' bounds: 1e-12, and float round-off for FP32
    assert rel_l2(want[0], o.as_deviation(f), geom.solid == 0) < {"fp64": 1e-12, "fp32": 3e-6}[precision]
