"""Two time steps per launch (march3d.hpp) on boxes that the routing rule gives
to it, asserted here box by box: every kind of walls, both lattices and both
storages, with ragged columns, rows and segments.  lbm_step(n) against
lbm_step(1) repeated, which always launches one step, bit for bit."""
import numpy as np
import pytest
import torch

import routes
from paper_2201_11330_amd import lbm
from paper_2201_11330_amd import workloads as W
from parity_utils import inputs

pytestmark = pytest.mark.gpu

FORCE = (1e-5, -2e-5, 3e-6)
NONE = (0, 0, 0)

CASES = [
    # lattice, dims, storage, bc, force, solid, compressible
    (W.D3Q19, (129, 141, 130), "f64", (2, 1, 1), FORCE, None, True),
    (W.D3Q19, (257, 92, 122), "f64", (1, 2, 2), NONE, None, False),
    (W.D3Q19, (257, 92, 121), "f64", (3, 1, 0), FORCE, None, False),
    (W.D3Q19, (258, 105, 121), "f64", (0, 0, 3), FORCE, "sphere", True),
    (W.D3Q19, (257, 105, 121), "f64", (0, 1, 0), FORCE, "sphere", False),
    (W.D3Q19, (257, 117, 101), "f64", (0, 0, 0), NONE, "random", False),
    (W.D3Q27, (193, 100, 117), "f64", (0, 1, 2), FORCE, None, False),
    (W.D3Q27, (257, 90, 133), "f64", (3, 0, 0), NONE, None, True),
    (W.D3Q27, (257, 90, 210), "f64", (0, 1, 0), FORCE, "random", False),
    (W.D3Q27, (257, 90, 210), "f64", (0, 3, 0), NONE, "sphere", True),
    (W.D3Q19, (129, 118, 97), "f32", (0, 0, 0), FORCE, None, False),
    (W.D3Q19, (128, 128, 96), "f32", (0, 0, 0), NONE, None, True),
    (W.D3Q19, (257, 118, 131), "f32", (0, 1, 0), FORCE, None, False),
    (W.D3Q19, (257, 130, 160), "f32", (2, 1, 0), NONE, None, True),
    (W.D3Q19, (257, 130, 140), "f32", (0, 3, 1), FORCE, "sphere", False),
    (W.D3Q19, (257, 130, 160), "f32", (0, 1, 0), FORCE, "random", True),
    (W.D3Q27, (130, 98, 99), "f32", (0, 0, 0), FORCE, None, False),
]


def _id(c):
    return "Q%d-%s-%s-bc%s-%s%s" % ({1: 19, 2: 27}[c[0]], "x".join(map(str, c[1])), c[2],
                                    "".join(map(str, c[3])), c[5] or "none", "-comp" if c[6] else "")


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_two_step_launches_equal_one_step_launches(case):
    lattice, dims, storage, bc, force, kind, comp = case
    print(_id(case), flush=True)
    assert routes.march(lattice, dims, storage, bc, kind is not None, comp)
    rho, u, _ = inputs(lattice, dims, "channel", seed=37, noise_amp=0, bc=bc, U0=0.03)
    solid = None
    if kind == "sphere":
        solid = W.sphere_mask(dims, tuple(n / 2.0 + 0.3 for n in dims), min(dims) / 4.0)
    elif kind == "random":
        solid = (np.random.default_rng(9).random(dims[::-1]) < 0.05).astype(np.uint8)
    if solid is not None:
        u[:, solid.astype(bool)] = 0.0
    sims = []
    for _ in range(2):
        sim = lbm.LBM(lattice, *dims, 0.7, force=force, bc=bc, storage=storage, compressible=comp)
        if solid is not None:
            sim.set_solid(solid)
        sim.init_equilibrium(rho, u)
        sims.append(sim)
    two, one = sims
    for n in (2, 5):
        two.step(n)
        for _ in range(n):
            one.step(1)
        assert torch.equal(two.get_populations(), one.get_populations())
    two.close()
    one.close()
