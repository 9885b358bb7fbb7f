"""Launches of several steps of D2Q9 boxes (regions, strips) on boxes that the
routing rule gives to them, asserted here launch by launch: every kind of
strips, with 16-bit storage too, between walls and around obstacles, and the
step counts that split a launch.  lbm_step(n) against lbm_step(1) repeated,
which always launches one step, bit for bit."""
import numpy as np
import pytest
import torch

import routes
from paper_2201_11330_amd import lbm
from paper_2201_11330_amd import workloads as W
from parity_utils import inputs

pytestmark = pytest.mark.gpu

S4, S8 = [(4, "strips")], [(8, "strips")]
CASES = [
    # dims, storage, bc, mask, compressible, launches of lbm_step: columns
    # and rows that do not fill strips and segments, and a second strip that
    # wraps (nx = 230, 256)
    ((1500, 1400), "f64", (0, 0, 0), False, False, S4 + S4 + [(3, "32x4")]),
    ((230, 9200), "f64", (0, 0, 0), False, True, S4 + [(3, "32x4")]),
    ((256, 8200), "f32", (0, 0, 0), False, False, S4 + [(1, "one")]),
    ((2900, 2900), "f32", (0, 0, 0), False, True, S8 + [(4, "32x4"), (2, "32x4")]),
    ((2100, 2000), "f16", (0, 0, 0), False, False, S4 + S4 + [(1, "one"), (1, "one")]),
    ((230, 18300), "f16", (0, 0, 0), False, True, S4 + S4),
    ((2100, 2000), "bf16", (0, 0, 0), False, True, S4 + [(1, "one")]),
    ((256, 16500), "bf16", (0, 0, 0), False, False, S4 + S4),
    ((2100, 2000), "e4m11", (0, 0, 0), False, False, S4 + S4 + [(1, "one")]),
    ((230, 18300), "e4m11", (0, 0, 0), False, False, S4),
    ((2000, 1600), "f16", (0, 0, 0), True, False, S4 + S4 + [(1, "one")]),
    ((230, 13700), "f16", (0, 3, 0), True, False, S4 + S4),
    ((2000, 1600), "bf16", (2, 1, 0), True, True, S4 + [(1, "one")]),
    ((230, 13700), "bf16", (0, 3, 0), True, False, S4),
    ((2900, 2900), "e4m11", (0, 1, 0), True, False, S4 + [(1, "one")]),
    ((2000, 1600), "f64", (0, 3, 0), False, True, S4 + [(3, "32x4")]),
    # halves and fours of six-step boxes; regions of four in every storage
    # that takes them
    ((700, 690), "f64", (0, 0, 0), False, False, [(6, "32x6"), (4, "32x4"), (4, "32x4")]),
    ((700, 690), "f16", (0, 0, 0), False, True, [(4, "32x4"), (4, "32x4")]),
    ((510, 520), "bf16", (0, 1, 0), False, False, [(4, "32x6"), (4, "32x6")]),
    ((510, 520), "f16", (0, 1, 0), False, True, [(5, "32x6"), (4, "32x6")]),
    ((510, 520), "f16", (0, 1, 0), True, True, [(6, "32x6"), (3, "32x6")]),
    ((153, 636), "e4m11", (0, 1, 0), False, True, [(6, "32x6"), (2, "32x6")]),
    ((400, 390), "e4m11", (0, 3, 0), False, False, [(6, "32x6"), (6, "32x6"), (1, "one")]),
    ((1030, 1024), "f32", (0, 0, 0), False, False, [(4, "32x4"), (4, "32x4"), (2, "32x4")]),
    ((1030, 1024), "f16", (0, 0, 0), False, True, [(4, "32x4"), (1, "one"), (1, "one")]),
    ((1030, 1020), "bf16", (0, 1, 0), False, True, [(4, "32x4"), (1, "one")]),
    ((1010, 1020), "e4m11", (0, 1, 0), True, False, [(4, "32x4"), (4, "32x4"), (1, "one")]),
    ((510, 520), "e4m11", (0, 3, 0), True, True, [(6, "32x6"), (1, "one")]),
    # a column and a row of blocks, tiles of blocks narrower than the XCD tile
    ((9, 4100), "f64", (0, 0, 0), False, False, [(8, "32x8"), (3, "32x8")]),
    ((30, 4100), "f32", (0, 1, 0), False, False, [(6, "32x6"), (5, "32x6")]),
    ((4100, 20), "f64", (0, 1, 0), False, True, [(6, "32x6"), (2, "32x6")]),
]


def _id(c):
    return "%dx%d-%s-bc%s%s%s" % (c[0] + (c[1], "".join(map(str, c[2])), "-mask" if c[3] else "",
                                          "-comp" if c[4] else ""))


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_launches_of_several_steps_equal_one_step_launches(case):
    dims, storage, bc, mask, comp, launches = case
    print(_id(case), flush=True)
    n = sum(k for k, _ in launches)
    assert routes.box_2d(dims, storage, any(bc), mask, comp, n) == launches
    rho, u, _ = inputs(W.D2Q9, dims + (1,), "channel", seed=43, noise_amp=0, bc=bc, U0=0.03)
    solid = None
    if mask:
        solid = (np.random.default_rng(7).random((1,) + dims[::-1]) < 0.08).astype(np.uint8)
        u[:, solid.astype(bool)] = 0.0
    sims = []
    for _ in range(2):
        sim = lbm.LBM(lbm.D2Q9, *dims, 1, 0.7, force=(1e-5, -2e-5, 0), bc=bc, storage=storage, compressible=comp)
        if mask:
            sim.set_solid(solid)
        sim.init_equilibrium(rho, u)
        sims.append(sim)
    many, one = sims
    many.step(n)
    for _ in range(n):
        one.step(1)
    assert many.steps_taken == one.steps_taken == n
    assert torch.equal(many.get_populations(), one.get_populations())
    many.close()
    one.close()
