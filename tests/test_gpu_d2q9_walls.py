"""Several D2Q9 time steps per launch between walls and around obstacles
(regions of fused2d.hpp, strips of stream2d.hpp), and launches of fewer than
four steps: lbm_step(n) against lbm_step(1) repeated, which always launches
one step.  The states agree bit for bit."""
import numpy as np
import pytest
import torch

from paper_2201_11330_amd import lbm
from paper_2201_11330_amd import workloads as W
from parity_utils import inputs, rel_err, run_oracle

pytestmark = pytest.mark.gpu

# Every region: 24 x 24 (boxes smaller than it among them), 32 x 32 with
# eight, six (in XCD-aware tiles and on a plain grid) and four steps; strips
# (periodic 2^21 nodes and more) with ragged columns and rows.
DIMS = [(7, 5), (40, 30), (130, 97), (200, 170), (260, 250), (300, 270), (600, 500), (1500, 1400), (230, 9200)]
BCS = [(0, 0, 0), (0, 1, 0), (2, 1, 0), (1, 2, 0), (0, 3, 0), (3, 1, 0)]


def _sim(dims, bc, storage, mask, comp, graph=False):
    nx, ny = dims
    sim = lbm.LBM(lbm.D2Q9, nx, ny, 1, 0.7, force=(1e-5, -2e-5, 0), bc=bc, storage=storage,
                  compressible=comp, graph=graph)
    rho, u, _ = inputs(W.D2Q9, (nx, ny, 1), "channel", seed=41, noise_amp=0, bc=bc, U0=0.03)
    solid = None
    if mask:
        solid = (np.random.default_rng(7).random((1, ny, nx)) < 0.08).astype(np.uint8)
        sim.set_solid(solid)
        u[:, solid.astype(bool)] = 0.0
    sim.init_equilibrium(rho, u)
    return sim, rho, u, solid


@pytest.mark.parametrize("storage,comp", [("f64", False), ("f64", True), ("f32", False), ("f16", True),
                                          ("e4m11", False)])
@pytest.mark.parametrize("mask", [False, True], ids=["axes", "mask"])
@pytest.mark.parametrize("bc", BCS, ids=lambda b: "bc" + "".join(map(str, b)))
@pytest.mark.parametrize("dims", DIMS, ids=lambda d: f"{d[0]}x{d[1]}")
def test_multi_step_launches_equal_one_step_launches(dims, bc, mask, storage, comp):
    print(dims, bc, mask, storage, comp, flush=True)
    many = _sim(dims, bc, storage, mask, comp)[0]
    one = _sim(dims, bc, storage, mask, comp)[0]
    for n in (4, 3, 10):
        many.step(n)
        for _ in range(n):
            one.step(1)
        assert many.steps_taken == one.steps_taken
        assert torch.equal(many.get_populations(), one.get_populations())
    many.close()
    one.close()


@pytest.mark.parametrize("bc,mask", [((2, 1, 0), True), ((0, 3, 0), False)])
def test_multi_step_launches_against_the_oracle(bc, mask):
    dims = (130, 97)
    sim, rho, u, solid = _sim(dims, bc, "f64", mask, False)
    sim.step(14)
    f_ref = run_oracle(W.D2Q9, dims + (1,), 0.7, (1e-5, -2e-5, 0), bc, rho, u, None, 14, solid=solid)[0]
    assert rel_err(sim.get_populations().cpu().numpy(), f_ref) <= 1e-12
    sim.close()


def test_graph_replays_between_walls():
    """Captured launches of four steps between walls, step counts that leave
    remainders, and eager work between the replays."""
    graph = _sim((130, 97), (0, 1, 0), "f64", True, False, graph=True)[0]
    eager = _sim((130, 97), (0, 1, 0), "f64", True, False)[0]
    for n in (3, 35, 6, 64, 37, 1, 32):
        graph.step(n)
        eager.step(n)
        assert torch.equal(graph.get_populations(), eager.get_populations())
        assert graph.wall_force() == eager.wall_force()
    graph.close()
    eager.close()


# Between walls strips are taken from 3 * 2^20 nodes up.
@pytest.mark.parametrize("bc,mask", [((0, 1, 0), False), ((2, 1, 0), True), ((0, 3, 0), False)])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("dims", [(230, 13700), (2000, 1600)], ids=lambda d: f"{d[0]}x{d[1]}")
def test_strips_between_walls_equal_one_step_launches(dims, bc, mask, storage):
    test_multi_step_launches_equal_one_step_launches(dims, bc, mask, storage, False)


# Graphs of pairs of eight- and of six-step launches.
@pytest.mark.parametrize("dims", [(97, 120), (260, 250), (300, 270)], ids=lambda d: f"{d[0]}x{d[1]}")
def test_graph_replays_of_regions(dims):
    graph = _sim(dims, (0, 1, 0), "f64", True, False, graph=True)[0]
    eager = _sim(dims, (0, 1, 0), "f64", True, False)[0]
    for n in (3, 45, 10, 64):
        graph.step(n)
        eager.step(n)
        assert torch.equal(graph.get_populations(), eager.get_populations())
    graph.close()
    eager.close()


# Periodic boxes of 2^22 nodes (FP64) and 2^23 (FP32): strips of eight steps,
# ragged columns and rows, a strip wider than the part it stores (nx = 230).
@pytest.mark.parametrize("dims,storage,comp", [((2100, 2000), "f64", False), ((230, 18300), "f64", True),
                                               ((2900, 2900), "f32", False)])
def test_eight_step_strips_equal_one_step_launches(dims, storage, comp):
    many = _sim(dims, (0, 0, 0), storage, False, comp)[0]
    one = _sim(dims, (0, 0, 0), storage, False, comp)[0]
    for n in (8, 13, 23):
        many.step(n)
        for _ in range(n):
            one.step(1)
        assert torch.equal(many.get_populations(), one.get_populations())
    many.close()
    one.close()


def test_graph_replays_of_eight_step_strips():
    graph = _sim((2100, 2000), (0, 0, 0), "f64", False, False, graph=True)[0]
    eager = _sim((2100, 2000), (0, 0, 0), "f64", False, False)[0]
    for n in (3, 45, 10, 64):
        graph.step(n)
        eager.step(n)
        assert torch.equal(graph.get_populations(), eager.get_populations())
    graph.close()
    eager.close()
