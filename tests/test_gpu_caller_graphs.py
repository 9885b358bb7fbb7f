"""Calls captured by the caller into HIP graphs of its own (torch.cuda.graph
on the context's stream) and replayed: every replay of an even number of
steps advances the state, whatever eager steps, new states and replays of
other graphs of the context lie between, as long as the step count has the
capture's parity at each replay.  Reference: a context that only makes
lbm_step(1) calls (one step per launch), bit for bit."""
import pytest
import torch

from paper_2201_11330_amd import lbm
from paper_2201_11330_amd import workloads as W
from parity_utils import inputs

pytestmark = pytest.mark.gpu

# Boxes that take launches of two (3D), eight, six and four steps (regions
# and strips), one that takes one-step launches, and the in-place pattern.
CASES = [
    # lattice, dims, storage, bc, solid, aa, steps per replay
    (W.D3Q19, (64, 64, 64), "f64", (0, 0, 0), False, False, 2),
    (W.D3Q19, (129, 118, 97), "f32", (0, 0, 0), False, False, 6),
    (W.D3Q27, (257, 90, 210), "f64", (0, 1, 0), True, False, 4),
    (W.D2Q9, (128, 128, 1), "f64", (0, 0, 0), False, False, 8),
    (W.D2Q9, (260, 250, 1), "f16", (0, 1, 0), True, False, 2),
    (W.D2Q9, (300, 270, 1), "f64", (0, 0, 0), False, False, 14),
    (W.D2Q9, (1500, 1400, 1), "f64", (0, 0, 0), False, False, 4),
    (W.D2Q9, (2100, 2000, 1), "f64", (0, 0, 0), False, False, 8),
    (W.D3Q19, (20, 14, 11), "f64", (0, 0, 0), False, False, 2),
    (W.D3Q19, (64, 64, 64), "f64", (0, 0, 0), False, True, 2),
]


def _id(c):
    return "%s-%s-%s-bc%s%s%s-n%d" % ({W.D2Q9: "Q9", W.D3Q19: "Q19", W.D3Q27: "Q27"}[c[0]],
                                      "x".join(map(str, c[1])), c[2], "".join(map(str, c[3])),
                                      "-solid" if c[4] else "", "-aa" if c[5] else "", c[6])


def _sim(case, stream):
    lattice, dims, storage, bc, solid, aa, _ = case
    sim = lbm.LBM(lattice, *dims, 0.7, bc=bc, storage=storage, aa=aa, stream=stream)
    rho, u, _ = inputs(lattice, dims, "channel", seed=51, noise_amp=0, bc=bc, U0=0.03)
    if solid:
        mask = torch.rand(dims[::-1], generator=torch.Generator().manual_seed(3)) < 0.05
        sim.set_solid(mask)
        u[:, mask.numpy()] = 0.0
    sim.init_equilibrium(rho, u)
    return sim, rho, u


def _capture(stream, fn):
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        fn()
    return graph


@pytest.mark.parametrize("before", [0, 2, 3], ids=lambda b: f"after{b}")
@pytest.mark.parametrize("case", CASES, ids=_id)
def test_replays_of_captured_calls(case, before):
    print(_id(case), before, flush=True)
    n = case[6]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim, rho, u = _sim(case, stream)
        one = _sim(case, stream)[0]
        monitor = torch.empty(4, dtype=torch.float64, device="cuda")
        fields = (torch.empty(case[1][::-1], dtype=torch.float64, device="cuda"),
                  torch.empty((3,) + case[1][::-1], dtype=torch.float64, device="cuda"))
        f = torch.empty((sim.Q,) + case[1][::-1], dtype=torch.float64, device="cuda")

        def same(steps):
            for _ in range(steps):
                one.step(1)
            assert torch.equal(sim.get_populations(), one.get_populations())

        sim.step(before)
        same(before)

        def outputs():
            sim.reduce_noalloc(monitor)
            sim.moments(rho=fields[0], u=fields[1])
            lbm.check(lbm.lib().lbm_get_populations(sim._h, lbm._ptr(f)), "lbm_get_populations")

        read = _capture(stream, outputs)
        step = _capture(stream, lambda: sim.step(n))

        def replay():
            step.replay()
            same(n)
            read.replay()
            red = one.reduce()
            assert monitor.tolist() == [red["mass"], red["ke"], red["umax"], 0.0]
            assert torch.equal(f, one.get_populations())
            assert all(torch.equal(a, b) for a, b in zip(fields, one.moments()))

        for _ in range(3):
            replay()
        for k in (2, 4, 6):  # eager steps between replays
            sim.step(k)
            same(k)
            replay()
        if before % 2 == 0:  # a new state between replays
            for s in (sim, one):
                s.init_equilibrium(rho, u)
            replay()
            replay()
            for s in (sim, one):
                s.step(1)
                s.step(3)
            replay()
    torch.cuda.synchronize()
    sim.close()
    one.close()
