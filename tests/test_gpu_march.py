"""Two time steps per launch on 3D boxes (march3d.hpp): lbm_step(n) of a
two-lattice D3Q19 or D3Q27 box in FP64 or FP32 storage against lbm_step(1)
repeated, which always launches one step.  The arithmetic per node is the
same, so the states agree bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2201_11330_amd import lbm
from paper_2201_11330_amd import workloads as W
from parity_utils import inputs, rel_err

pytestmark = pytest.mark.gpu

FORCE = (1e-5, -2e-5, 3e-6)

# Boxes above the sizes that take the launches: tiles of 64 columns with a
# remainder of 1, 2 or none, rows that do not fill the last tile, segments
# of unequal length, planes that are whole tiles of the stored state
# (64 x 64) and planes that are not, rows shorter than a tile (33, 40).
CASES = [
    # lattice, dims, storage, bc, force, solid, compressible
    (W.D3Q19, (64, 64, 64), "f64", (0, 0, 0), (0, 0, 0), None, False),
    (W.D3Q19, (66, 70, 60), "f64", (0, 0, 0), FORCE, None, False),
    (W.D3Q19, (129, 27, 80), "f64", (0, 0, 0), FORCE, None, True),
    (W.D3Q19, (40, 14, 481), "f64", (0, 0, 0), FORCE, None, False),
    (W.D3Q19, (257, 260, 4), "f64", (0, 0, 0), (0, 0, 0), None, False),
    (W.D3Q19, (100, 75, 75), "f64", (0, 1, 0), FORCE, None, False),
    (W.D3Q19, (129, 66, 63), "f64", (2, 1, 1), FORCE, None, True),
    (W.D3Q19, (97, 90, 61), "f64", (1, 2, 2), (0, 0, 0), None, False),
    (W.D3Q19, (100, 75, 75), "f64", (0, 3, 0), FORCE, None, False),
    (W.D3Q19, (97, 90, 61), "f64", (3, 1, 0), FORCE, None, False),
    (W.D3Q19, (97, 90, 61), "f64", (0, 0, 3), FORCE, "sphere", True),
    (W.D3Q19, (100, 75, 75), "f64", (0, 1, 0), FORCE, "sphere", False),
    (W.D3Q19, (129, 66, 63), "f64", (0, 0, 0), (0, 0, 0), "random", False),
    (W.D3Q27, (66, 70, 60), "f64", (0, 0, 0), FORCE, None, False),
    (W.D3Q27, (130, 91, 90), "f64", (0, 1, 2), FORCE, None, False),
    (W.D3Q27, (130, 91, 90), "f64", (3, 0, 0), (0, 0, 0), None, True),
    (W.D3Q27, (130, 91, 90), "f64", (0, 1, 0), FORCE, "random", False),
    (W.D3Q19, (65, 105, 97), "f32", (0, 0, 0), FORCE, None, False),
    (W.D3Q19, (128, 64, 81), "f32", (0, 0, 0), (0, 0, 0), None, True),
    (W.D3Q19, (129, 128, 128), "f32", (0, 1, 0), FORCE, None, False),
    (W.D3Q19, (129, 128, 128), "f32", (0, 3, 1), FORCE, "sphere", False),
    (W.D3Q27, (65, 105, 97), "f32", (0, 0, 0), FORCE, None, False),
]


def _solid(kind, dims):
    if kind is None:
        return None
    nx, ny, nz = dims
    if kind == "sphere":
        return W.sphere_mask(dims, (nx / 2.0, ny / 2.0 + 0.3, nz / 2.0), min(dims) / 4.0)
    return (np.random.default_rng(9).random((nz, ny, nx)) < 0.05).astype(np.uint8)


def _id(c):
    return "Q%d-%s-%s-bc%s-%s%s" % ({1: 19, 2: 27}[c[0]], "x".join(map(str, c[1])), c[2],
                                    "".join(map(str, c[3])), c[5] or "none", "-comp" if c[6] else "")


def _sim(case, graph=False):
    lattice, dims, storage, bc, force, kind, comp = case
    sim = lbm.LBM(lattice, *dims, 0.7, force=force, bc=bc, storage=storage, compressible=comp, graph=graph)
    solid = _solid(kind, dims)
    if solid is not None:
        sim.set_solid(solid)
    rho, u, _ = inputs(lattice, dims, "channel", seed=31, noise_amp=0, bc=bc, U0=0.03)
    if solid is not None:
        u[:, solid.astype(bool)] = 0.0
    sim.init_equilibrium(rho, u)
    return sim, rho, u, solid


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_two_step_launches_equal_one_step_launches(case):
    print(_id(case), flush=True)
    two, rho, u, solid = _sim(case)
    one = _sim(case)[0]
    for n in (2, 5):
        two.step(n)
        for _ in range(n):
            one.step(1)
        assert two.steps_taken == one.steps_taken
        assert torch.equal(two.get_populations(), one.get_populations())
    two.close()
    one.close()


@pytest.mark.parametrize("case", [CASES[1], CASES[11]], ids=_id)
def test_two_step_launches_against_the_oracle(case):
    lattice, dims, _, bc, force, _, comp = case
    print(_id(case), flush=True)
    sim, rho, u, solid = _sim(case)
    sim.step(6)
    ref = oracle.Sim(lattice, *dims, tau=0.7, force=force, bc=bc, compressible=comp)
    if solid is not None:
        ref.set_solid(solid)
    ref.init_equilibrium(rho, u)
    ref.step(6)
    assert rel_err(sim.get_populations().cpu().numpy(), ref.get_populations()) <= 1e-12
    sim.close()
    ref.close()


def test_graph_replays_of_two_step_launches():
    """32 captured steps are 16 launches of two; a step count that is not a
    multiple of four, before and between replays, leaves the buffers where
    the next replay expects them.  Replays with eager work of the same
    context between them."""
    case = CASES[0]
    graph = _sim(case, graph=True)[0]
    eager = _sim(case)[0]
    for n in (3, 35, 2, 64, 33, 1, 32):
        graph.step(n)
        eager.step(n)
        assert torch.equal(graph.get_populations(), eager.get_populations())
        assert graph.reduce() == eager.reduce()
    graph.close()
    eager.close()


@pytest.mark.parametrize("n,k", [(6, 3), (8, 2), (4, 1)])
def test_checkpoints_of_two_step_launches(n, k):
    """The states that lbm_forward_record keeps are those of one-step
    launches, wherever the two-step launches have left the current buffer.
    (A box of whole tiles: the stored state has no padding.)"""
    case = CASES[0]
    two = _sim(case)[0]
    one = _sim(case)[0]
    ckpt = two.forward_record(n, k).view(n // k, -1)
    for s in range(n // k):
        assert torch.equal(one.forward_record(1, 1), ckpt[s])  # the state before the step
        for _ in range(k - 1):
            one.step(1)
    assert torch.equal(two.get_populations(), one.get_populations())
    two.close()
    one.close()
