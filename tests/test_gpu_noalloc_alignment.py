"""lbm_reduce_noalloc into results at any address, as a copy takes them: also
where the destination is not aligned for FP64 stores."""
import ctypes

import pytest
import torch

from paper_2201_11330_amd import lbm
from paper_2201_11330_amd import workloads as W
from parity_utils import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1, 4, 8, 12])
def test_result_at_any_address(offset):
    print(offset, flush=True)
    rho, u, _ = inputs(W.D3Q19, (20, 14, 11), "channel", seed=71, noise_amp=0)
    sim = lbm.LBM(lbm.D3Q19, 20, 14, 11, 0.7)
    sim.init_equilibrium(rho, u)
    sim.step(3)
    raw = torch.full((64,), 0xA5, dtype=torch.uint8, device="cuda")
    for _ in range(2):
        lbm.check(lbm.lib().lbm_reduce_noalloc(sim._h, ctypes.c_void_p(raw.data_ptr() + offset)), "lbm_reduce_noalloc")
        torch.cuda.synchronize()
        host = bytes(raw.cpu().tolist())
        red = sim.reduce()
        got = (ctypes.c_double * 4).from_buffer_copy(host[offset:offset + 32])
        assert list(got) == [red["mass"], red["ke"], red["umax"], 0.0]
        assert set(host[:offset] + host[offset + 32:]) == {0xA5}
        sim.step(2)
    sim.close()
