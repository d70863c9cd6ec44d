"""Which path a step takes, and the paths of launches on tiles that need more
than an ordinary obstacle (GPU): regions with more cut links than a block has
threads, in every variant of the kernel; domains whose regions exceed what a
block carries; recorded runs; objectives whose window opens in mid-run; the raw
state.  Each against single steps (LBM_DEBUG=1), bit for bit."""

import numpy as np
import pytest

from gpu_util import require_gpu
from test_gpu_tiles import CASES
from workloads import configs, states
from workloads import geometry as G
from workloads.velocities import VELOCITIES

pytestmark = pytest.mark.gpu
THREADS = 512            # of a block on tiles

RATES = {"D2Q9": configs.d2q9_rates(0.62), "D3Q15": configs.d3q15_paper_rates(1.2),
         "D3Q19": configs.d3q19_rates(0.7)}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def scattered(lattice, shape, share, x_bc="periodic", seed=1):
    """Solid nodes drawn one by one: the cut links lie everywhere."""
    rng = np.random.default_rng(seed)
    nx, ny, nz = shape
    n = np.arange(nx * ny * nz)
    x, y, z = n % nx, (n // nx) % ny, n // (nx * ny)
    solid = rng.random(n.size) < share
    if x_bc == "outflow":
        solid[x == 0] = True
    node, direction = [], []
    for i, e in enumerate(VELOCITIES[lattice]):
        sx = x - e[0]
        sx = np.clip(sx, 0, nx - 1) if x_bc == "outflow" else sx % nx
        src = sx + nx * ((y - e[1]) % ny + ny * ((z - (e[2] if len(e) == 3 else 0)) % nz))
        at = np.nonzero(~solid & solid[src])[0]
        node.append(at)
        direction.append(np.full(at.size, i))
    node, direction = np.concatenate(node).astype(np.int64), np.concatenate(direction).astype(np.int8)
    L, D = node.size, len(VELOCITIES[lattice][0])
    return G.Geometry(lattice, shape, solid.astype(np.uint8), node, direction, 1.0 - rng.random(L),
                      0.01 * rng.normal(size=(L, D)), np.ones(L, np.int32), x_bc, {})


def solver(geom, precision, kw):
    from paper_1712_08288_amd import binding
    sv = binding.solver_for(geom, RATES[geom.lattice], g=kw.get("g"), dp=kw.get("dp", 0.0),
                            l_rule="gamma2", b=kw.get("b", 1.0),
                            two_node=kw.get("two_node", False), precision=precision)
    sv.set_wall_decay(kw.get("decay", 1.0))
    return sv


def start(geom):
    df = states.random_deviation(len(RATES[geom.lattice]), geom.n_nodes, seed=3)
    if geom.x_bc == "outflow":
        df = states.outlet_consistent(df, geom.shape, VELOCITIES[geom.lattice])
    return df


def both(monkeypatch, geom, precision, kw, run):
    """run(solver) on tiles and in single steps; the results must be equal."""
    out = []
    for mode in ("0", "1"):
        monkeypatch.setenv("LBM_DEBUG", mode)
        sv = solver(geom, precision, kw)
        if mode == "1":
            assert sv.tile_plan(33) == (1, 0, 0)
        sv.init_deviation(start(geom))
        out.append(run(sv))
        sv.close()
    for k, (a, b) in enumerate(zip(*out)):
        assert np.array_equal(a, b, equal_nan=True), k


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_the_compared_domains_take_tiles(name, precision):
    make, kw = CASES[name]
    sv = solver(make(), precision, kw)
    steps, blocks, links = sv.tile_plan(33)
    sv.close()
    assert steps > 1 and blocks >= 1 and links >= 1


# shares of solid nodes that give a region of each precision 512 to 1024 links
DENSE = {
    "plain": ("D2Q9", (300, 200, 1), (0.12, 0.055), {}),
    "decay": ("D2Q9", (300, 200, 1), (0.12, 0.055), dict(decay=0.97, b=0.7)),
    "two_node": ("D2Q9", (300, 200, 1), (0.12, 0.055), dict(two_node=True)),
    "seam": ("D2Q9", (301, 201, 1), (0.12, 0.055), dict(dp=1e-3, x_bc="pressure")),
    "two_node_seam": ("D2Q9", (301, 201, 1), (0.12, 0.055), dict(dp=1e-3, x_bc="pressure", two_node=True)),
    "outflow": ("D2Q9", (300, 200, 1), (0.12, 0.055), dict(x_bc="outflow")),
    "d3q15": ("D3Q15", (2, 60, 60), (0.2, 0.1), {}),
    "d3q19_two_node": ("D3Q19", (2, 60, 60), (0.16, 0.05), dict(two_node=True)),
}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(DENSE))
def test_regions_with_more_links_than_threads(monkeypatch, name, precision):
    lattice, shape, share, kw = DENSE[name]
    geom = scattered(lattice, shape, share[precision == "fp32"], kw.get("x_bc", "periodic"))

    def run(sv):
        got = []
        for n in (9, 20):
            sv.set_objective("force_x", 1, sv.time + 2, sv.time + n - 1)
            sv.step(n)
            got += [sv.distribution(), np.array(sv.objective()), sv.force(2)]
        return got

    sv = solver(geom, precision, kw)
    steps, _, links = sv.tile_plan(33)
    sv.close()
    assert steps > 1 and THREADS < links <= 2 * THREADS, (steps, links)
    both(monkeypatch, geom, precision, kw, run)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_regions_beyond_a_blocks_links_take_single_steps(monkeypatch, precision):
    """Every other node solid: no plan's regions hold their links."""
    geom = scattered("D2Q9", (300, 200, 1), 0.5)
    sv = solver(geom, precision, {})
    assert sv.tile_plan(33) == (1, 0, 0)
    sv.close()
    both(monkeypatch, geom, precision, {}, lambda sv: [sv.step(33), sv.distribution()][1:])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["tiles", "two_node_seam", "outflow", "pipe"])
def test_recorded_runs(monkeypatch, name, precision):
    """Tiles up to the recorded last step of a segment."""
    make, kw = CASES[name]
    geom = make()

    def run(sv):
        sv.set_rate_gradient(False)
        sv.set_objective("force_x", int(geom.tag.max()), 4, 19)
        sv.run_checkpointed(23, 9)
        sv.adjoint()
        gr = sv.grad()
        return [sv.distribution(), np.array(sv.objective()), gr["q"], gr["wall_u"], gr["g"]]

    both(monkeypatch, geom, precision, kw, run)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name,objective", [("tiles", "mean_ux"), ("pipe", "mean_ux"),
                                            ("seam", "pressure_drop"), ("two_node", "force_x")])
def test_windows_of_single_steps_in_mid_run(monkeypatch, name, objective, precision):
    """Objectives summed in single steps: tiles before and behind the window."""
    make, kw = CASES[name]
    geom = make()

    def run(sv):
        debug = sv.tile_plan(64)[0] == 1
        sv.set_objective(objective, int(geom.tag.max()), 11, 17)
        ahead = sv.tile_plan(64)[0]
        assert debug or 1 < ahead <= 11
        sv.step(14)
        assert sv.tile_plan(20)[0] == 1          # inside the window
        sv.step(20)
        assert debug or sv.tile_plan(64)[0] > 1
        return [sv.distribution(), np.array(sv.objective())]

    both(monkeypatch, geom, precision, kw, run)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["tiles", "two_node", "outflow", "pipe"])
def test_raw_state(monkeypatch, name, precision):
    """What single steps write into a state (LBM_DEBUG leaves NaN in the rest),
    and the run that goes on from it."""
    import torch
    make, kw = CASES[name]
    geom = make()
    dtype = {"fp64": torch.float64, "fp32": torch.float32}[precision]
    raw, end = [], []
    for mode in ("0", "1"):
        monkeypatch.setenv("LBM_DEBUG", mode)
        sv = solver(geom, precision, kw)
        sv.init_deviation(start(geom))
        sv.step(30)
        state = torch.empty(sv.state_bytes(), dtype=torch.uint8, device="cuda")
        sv.get_state(state)
        raw.append(state.cpu().view(dtype).numpy())
        sv.close()
        monkeypatch.setenv("LBM_DEBUG", "0")
        sv = solver(geom, precision, kw)
        sv.set_state(state, 30)
        sv.step(9)
        end.append(sv.distribution())
        sv.close()
    written = ~np.isnan(raw[1])
    assert written.sum() > geom.n_fluid and np.array_equal(raw[0][written], raw[1][written])
    assert np.array_equal(end[0], end[1], equal_nan=True)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_graph_replay_without_tiles(monkeypatch, precision):
    """A domain that has no plan replays captured loops of 64 steps: equal to
    single launches bit for bit across odd counts, new parameters and links
    (which make captured loops invalid), a drag window and what comes behind."""
    geom = G.random_spheres(40, 40, 40, 8, 4.0, 7.0, seed=31)
    runs = []
    for graph in (True, False):
        if graph:
            monkeypatch.delenv("LBM_GRAPH_STEPS", raising=False)
        else:
            monkeypatch.setenv("LBM_GRAPH_STEPS", "0")
        sv = solver(geom, precision, dict(g=(1e-5, 0, 0)))
        assert sv.tile_plan(200) == (1, 0, 0)
        sv.init_deviation(start(geom))
        sv.step(131)
        out = [sv.distribution()]
        sv.set_parameters(configs.d3q19_rates(0.8), (2e-5, 1e-6, 0))
        sv.step(64)
        out.append(sv.distribution())
        sv.update_links(geom.q * 0.97)
        sv.step(129)
        out.append(sv.distribution())
        sv.set_objective("force_x", 1, sv.time + 10, sv.time + 90)
        sv.step(200)
        out += [sv.distribution(), np.array(sv.objective())]
        sv.step(128)
        out += [sv.distribution(), np.array([sv.objective(), sv.time])]
        runs.append(out)
        sv.close()
    for k, (a, b) in enumerate(zip(*runs)):
        assert np.array_equal(a, b, equal_nan=True), k


# (elements of 4 bytes, many blocks; thin domains without links that do not wrap)
@pytest.mark.parametrize("make,precision,two", [
    (lambda: G.random_cylinders(1800, 1300, 300, 4.0, 7.0, seed=5), "fp32", 1),
    (lambda: G.random_cylinders(1800, 1300, 300, 4.0, 7.0, seed=5), "fp64", 2),
    (lambda: G.random_cylinders(640, 400, 60, 4.0, 7.0, seed=5), "fp32", 2),
    (lambda: G.empty("D3Q15", (64, 64, 4)), "fp32", 1),
    (lambda: G.empty("D3Q15", (4, 64, 64)), "fp32", 2),
    (lambda: scattered("D3Q15", (64, 64, 4), 0.02), "fp32", 2),
    (lambda: G.random_spheres(16, 16, 16, 2, 2.0, 3.0, seed=5), "fp64", 2)])
def test_calls_of_two_steps(make, precision, two):
    """One launch or two single steps, whichever is faster: the same state."""
    geom = make()
    ends = []
    for calls in ((2, 2, 2), (6,)):
        sv = solver(geom, precision, {})
        assert sv.tile_plan(2)[0] == two and sv.tile_plan(4)[0] > 1
        sv.init_deviation(start(geom))
        for n in calls:
            sv.step(n)
        ends.append(sv.distribution())
        sv.close()
    assert np.array_equal(*ends, equal_nan=True)
