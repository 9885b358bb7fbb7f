"""Initial states, populations and moments of 3D boxes on both orders of
work-items (rows, where few lanes idle, and node order): row lengths and
heights on both sides of the three quarters and seven eighths of busy lanes at
which the order changes, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2201_11330_amd import lbm
from paper_2201_11330_amd import workloads as W
from parity_utils import inputs

pytestmark = pytest.mark.gpu

# Busy lanes: all, 7/8, just below, 3/4, just below, few; rows of more than
# one workgroup.
DIMS = [(64, 8, 5), (56, 12, 4), (55, 12, 4), (48, 12, 4), (47, 12, 4), (33, 9, 5), (300, 3, 3), (448, 4, 3)]
def _e(lattice):
    e = [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1)]
    return np.array([v for v in e if lattice == W.D3Q27 or sum(c * c for c in v) <= 2], dtype=float)


@pytest.mark.parametrize("bc,mask", [((0, 0, 0), False), ((0, 1, 0), False), ((0, 3, 2), False), ((0, 0, 0), True)])
@pytest.mark.parametrize("dims", DIMS, ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("lattice", [W.D3Q19, W.D3Q27], ids=["Q19", "Q27"])
def test_initial_state_and_moments(lattice, dims, bc, mask):
    """FP64 against the oracle; a reduced storage started from the fields holds
    what it holds when the FP64 populations are set, bit for bit (both round
    the same FP64 values)."""
    print(lattice, dims, bc, mask, flush=True)
    force = (1e-5, -2e-5, 3e-5)
    rho, u, _ = inputs(lattice, dims, "channel", seed=61, noise_amp=0, bc=bc, U0=0.03)
    noise = W.population_noise(lattice, dims, 1e-4, seed=62)
    solid = None
    if mask:
        solid = (np.random.default_rng(5).random(dims[::-1]) < 0.1).astype(np.uint8)
        u[:, solid.astype(bool)] = 0.0
    ref = oracle.Sim(lattice, *dims, tau=0.7, force=force, bc=bc)
    if mask:
        ref.set_solid(solid)
    ref.init_equilibrium(rho, u, noise)
    f_ref = ref.get_populations()
    ref.close()
    fluid = f_ref[f_ref.shape[0] // 2] != 0
    f64 = None
    for storage in ("f64", "f32", "f16"):
        sim = lbm.LBM(lattice, *dims, 0.7, force=force, bc=bc, storage=storage)
        if mask:
            sim.set_solid(solid)
        sim.init_equilibrium(rho, u, noise)
        f = sim.get_populations().cpu().numpy()
        if storage == "f64":
            # About ten operations of values below 1 in both.
            f64 = f
            assert np.abs(f - f_ref).max() <= 1e-14
        sim.set_populations(f64)
        assert np.array_equal(sim.get_populations().cpu().numpy(), f)
        # Sums of up to 27 values below 1, in the arithmetic type and here.
        tol = 2 * 27 * (2.0 ** -53 if storage == "f64" else 2.0 ** -24)
        r, v = (t.cpu().numpy() for t in sim.moments())
        v_ref = np.tensordot(_e(lattice).T, f, 1) + 0.5 * np.array(force)[:, None, None, None]
        assert np.abs(r - f.sum(0)).max() <= tol
        assert np.abs(v - v_ref * fluid).max() <= tol
        sim.close()
