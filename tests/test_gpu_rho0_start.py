"""The check of the initial density where it is made on the host (a lone
lattice of at most 16384 nodes, the mean density of the collision drive) and
just beyond, on the device: values outside the EOS domain anywhere in the
field, the smallest value, and the drive's mean."""
import dataclasses

import numpy as np
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_parity import p_cfg
from test_gpu_rho0_check import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("drive", [False, True])
@pytest.mark.parametrize("nx,ny", [(64, 64), (128, 128), (16385, 1), (300, 90)])
def test_values_outside_the_domain(nx, ny, drive):
    cfg = p_cfg(nx, ny, a=0.25, Tr=0.75)
    if drive:
        cfg = dataclasses.replace(cfg, ax=1e-5, x_split=nx // 2)
    n = nx * ny
    for at in (0, n // 2, n - 1):
        for bad in (np.nan, np.inf, 0.0, 1.0):  # b rho / 4 = 1 at rho = 1
            r = np.full((ny, nx), 0.1)
            r.reshape(-1)[at] = bad
            with pytest.raises(lbm.LbmError) as e:
                lbm.Simulation(cfg, dev(r))
            assert e.value.status == lbm.ERR_EOS_DOMAIN


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("nx,ny", [(64, 64), (150, 130)])
def test_mean_density_of_the_drive(nx, ny, prec):
    """Left to the library and given: the same run."""
    rng = np.random.default_rng(7)
    r = 0.2 * (1 + 0.1 * rng.uniform(-1, 1, size=(ny, nx)))
    cfg = dataclasses.replace(p_cfg(nx, ny, a=0.25, Tr=0.75, precision=prec), ax=1e-3,
                              x_split=nx // 2)
    out = []
    for ave in (0.0, np.float64(sum(sorted(map(float, r.ravel()))) / r.size)):
        sim = lbm.Simulation(dataclasses.replace(cfg, rho_ave=float(ave)), dev(r))
        sim.step(20)
        out.append(sim.populations().cpu().numpy())
        sim.close()
    # the two means differ by the rounding of their sums, 19500 terms
    bound = 1e-9 if prec == lbm.FP64 else 1e-6
    assert np.max(np.abs(out[0] - out[1])) <= bound * 0.2
