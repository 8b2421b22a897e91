"""The check of the initial density on the device: a value outside the EOS
domain is found wherever it stands (first, last and middle node; fields of
one block, of several and of a remainder), alone and inside a batch, and the
smallest value, which sets the FP32 storage shift, is found at the ends."""
import numpy as np
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_parity import p_cfg, torch_dev

pytestmark = pytest.mark.gpu


def dev(r):
    import torch
    return torch.from_numpy(np.ascontiguousarray(r)).to(torch_dev())


@pytest.mark.parametrize("nx,ny", [(1, 1), (7, 5), (256, 8), (2049, 1), (257, 130)])
def test_values_outside_the_domain(nx, ny):
    cfg = p_cfg(nx, ny, a=0.25, Tr=0.75, precision=lbm.FP32_SHIFTED)
    good = np.full((ny, nx), 0.1)
    lbm.Simulation(cfg, dev(good)).close()
    n = nx * ny
    for at in {0, n // 2, n - 1}:
        for bad in (np.nan, np.inf, -np.inf, 0.0, -0.1, 1.0):  # b rho / 4 = 1 at rho = 1
            r = good.copy()
            r.reshape(-1)[at] = bad
            with pytest.raises(lbm.LbmError) as e:
                lbm.Simulation(cfg, dev(r))
            assert e.value.status == lbm.ERR_EOS_DOMAIN
            with pytest.raises(lbm.LbmError) as e:
                lbm.Batch([cfg, cfg, cfg], [dev(good), dev(r), dev(good)])
            assert e.value.status == lbm.ERR_EOS_DOMAIN


@pytest.mark.parametrize("nx,ny", [(7, 5), (2049, 1), (257, 130)])
@pytest.mark.parametrize("where", ["first", "last"])
def test_smallest_value_sets_the_shift(nx, ny, where):
    """The deviation from the reference, the smallest density rounded to 20
    bits, is stored in FP32: that node's density comes back to within those
    20 bits of itself, which a reference of the other nodes' size (0.3, a
    rounding of 2^-24 0.3 on 1e-6) would miss."""
    cfg = p_cfg(nx, ny, a=0.25, Tr=0.75, precision=lbm.FP32_SHIFTED)
    r = np.full((ny, nx), 0.3)
    at = 0 if where == "first" else nx * ny - 1
    r.reshape(-1)[at] = 1e-6
    sim = lbm.Simulation(cfg, dev(r))
    f = sim.populations().cpu().numpy().reshape(9, -1)[:, at].sum()
    sim.close()
    assert abs(f - 1e-6) <= 9 * 2.0 ** -24 * 1e-6
