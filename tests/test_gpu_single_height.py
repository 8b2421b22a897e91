"""Single steps beside two-step launches on a lattice whose segment height is
left to the library (they take segments of their own): odd counts and calls
for one step equal the same lattice with a given height bit for bit."""
import numpy as np
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_parity import fe_cfg, p_cfg
from test_gpu_patch import P_KW
from test_gpu_two_step import FE_TAU

pytestmark = pytest.mark.gpu


def run(cfg, rho0, chunks):
    import torch
    sim = lbm.Simulation(cfg, rho0)
    for n in chunks:
        sim.step(n)
    obs, fields = sim.observe(fields=True)
    f = sim.populations()
    info = sim.launch_info()
    sim.close()
    return obs, fields, f, info


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("model", ["P", "FE"])
@pytest.mark.parametrize("nx,ny", [(2100, 2003), (300, 14001), (30011, 141)])
def test_odd_counts(nx, ny, model, prec):
    import torch
    cfg = (p_cfg(nx, ny, a=0.25, Tr=0.75, precision=prec, **P_KW) if model == "P"
           else fe_cfg(nx, ny, a=0.25, Tr=0.75, tau=FE_TAU, precision=prec))
    g = torch.Generator(device="cuda:0").manual_seed(3)
    rho0 = 0.2 * (1 + 0.05 * (2 * torch.rand((ny, nx), generator=g, device="cuda:0",
                                             dtype=torch.float64) - 1))
    chunks = (1, 2, 1, 19, 3)
    a = run(cfg, rho0, chunks)
    b = run(cfg.with_launch(256, 64, 0), rho0, chunks)
    assert a[3]["steps_per_launch"] == 2 and b[3]["segment"] == 64
    assert a[0]["flags"] == b[0]["flags"] and a[0]["mass"] == b[0]["mass"]
    for x, y in zip(a[1], b[1]):
        assert torch.equal(x, y)
    assert torch.equal(a[2], b[2])
