"""lbm_wall_force on boxes that take its work-items through more than eight
nodes each (more than 8 * 2^18 nodes, no multiple of 2^18), with a mask and
without: against the sum over the links formed here from the exported
populations."""
import numpy as np
import pytest
import torch

from paper_2201_11330_amd import lbm
from paper_2201_11330_amd import workloads as W
from parity_utils import inputs

pytestmark = pytest.mark.gpu

CASES = [
    # lattice, dims, bc, mask, storage, aa
    (W.D3Q19, (131, 127, 131), (0, 1, 0), True, "f64", False),
    (W.D3Q19, (131, 127, 131), (2, 1, 0), False, "f64", False),
    (W.D3Q19, (131, 127, 131), (0, 2, 3), True, "f16", True),
    (W.D3Q19, (131, 127, 131), (0, 0, 1), False, "f64", True),
    (W.D3Q27, (67, 259, 130), (1, 0, 2), True, "f32", False),
    (W.D3Q27, (67, 259, 130), (3, 1, 0), False, "f64", True),
    (W.D2Q9, (1501, 1409, 1), (2, 3, 0), True, "f64", False),
    (W.D2Q9, (1501, 1409, 1), (1, 2, 0), False, "f16", True),
]


def _directions(lattice):
    if lattice == W.D2Q9:
        return [(x, y, 0) for x in (-1, 0, 1) for y in (-1, 0, 1)]
    e = [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1)]
    return [v for v in e if lattice == W.D3Q27 or sum(c * c for c in v) <= 2]


def _link_sum(f, dims, lattice, bc, solid):
    """Sum of 2 f_abar e_a over the links from fluid into walls, and the sum
    of the terms' magnitudes and their number."""
    nx, ny, nz = dims
    coords = torch.meshgrid(*(torch.arange(n, device="cuda") for n in (nz, ny, nx)), indexing="ij")[::-1]
    e = _directions(lattice)
    total, size, links = torch.zeros(3, dtype=torch.float64), 0.0, 0
    for a, v in enumerate(e):
        wall = torch.roll(solid, (-v[2], -v[1], -v[0]), (0, 1, 2)).clone()
        beyond_nodal = torch.zeros_like(solid)
        for d in range(3):
            t = coords[d] + v[d]
            out = (t < 0) | (t >= dims[d])
            if bc[d] == W.PERIODIC:
                continue
            wall |= out
            if bc[d] == 3:
                beyond_nodal |= out
        hit = wall & ~beyond_nodal & ~solid
        term = 2.0 * f[len(e) - 1 - a][hit]
        total += term.sum().cpu() * torch.tensor(v, dtype=torch.float64)
        size += float(term.abs().sum())
        links += int(hit.sum())
    return total.numpy(), size, links


@pytest.mark.parametrize("case", CASES, ids=lambda c: "Q%d-%s-bc%s%s-%s%s" % (
    {0: 9, 1: 19, 2: 27}[c[0]], "x".join(map(str, c[1])), "".join(map(str, c[2])), "-mask" if c[3] else "", c[4],
    "-aa" if c[5] else ""))
def test_wall_force_of_many_nodes_per_work_item(case):
    lattice, dims, bc, mask, storage, aa = case
    print(case, flush=True)
    assert dims[0] * dims[1] * dims[2] > 8 << 18
    force = (1e-5, -2e-5, 0.0 if lattice == W.D2Q9 else 3e-5)
    sim = lbm.LBM(lattice, *dims, 0.7, force=force, bc=bc, storage=storage, aa=aa)
    rho, u, _ = inputs(lattice, dims, "channel", seed=81, noise_amp=0, bc=bc, U0=0.03)
    solid = torch.zeros(dims[::-1], dtype=torch.bool)
    if mask:
        m = np.random.default_rng(11).random(dims[::-1]) < 0.02
        m[..., : dims[0] // 3] = False  # nodes without a wall, and many with
        sim.set_solid(m.astype(np.uint8))
        solid |= torch.from_numpy(m)
    for d in range(3):
        if bc[d] == W.SOLID_ENDS:
            solid.select(2 - d, 0).fill_(True)
            solid.select(2 - d, dims[d] - 1).fill_(True)
    u[:, solid.numpy()] = 0.0
    sim.init_equilibrium(rho, u)
    solid = solid.cuda()
    for n in (4, 1):  # both parities of the in-place pattern
        sim.step(n)
        ref, size, links = _link_sum(sim.get_populations(), dims, lattice, bc, solid)
        assert links > 1000
        # Any order of `links` additions.
        assert np.abs(np.array(sim.wall_force()) - ref).max() <= 2 * links * 2.0 ** -53 * size
    sim.close()
