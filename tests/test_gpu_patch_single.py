"""Large lattices on patches whose single steps go to the strips: calls for one
step and counts with a remainder of one, between patch launches, equal the
same lattice on explicit strips bit for bit."""
import dataclasses

import numpy as np
import pytest

from oracle import theory as th
from paper_2403_11167_amd import inputs, lbm
from test_gpu_parity import p_cfg
from test_gpu_patch import P_KW, same
from test_gpu_patch_general import channel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,prec", [(1500, 1401, lbm.FP64), (2003, 2001, lbm.FP32_SHIFTED)])
def test_channel(nx, ny, prec):
    cfg, rho0 = channel(nx, ny, "P", prec)
    _, info = same(cfg, rho0, (1, 1, 3, 1, 4, 7), walls=True)
    assert info["steps_per_launch"] > 1


def test_drive_switches_on_after_a_lone_step():
    """Step 3 is the first driven one: launches end before it, with one step
    left over."""
    nx, ny = 1500, 1401
    cfg = dataclasses.replace(p_cfg(nx, ny, a=0.25, Tr=0.8), ax=5e-4, x_split=nx // 2,
                              ax_from_step=3)
    rl, rv, _ = th.maxwell(cfg.eos, cfg.a, cfg.b, cfg.R, cfg.T)
    rho0 = inputs.droplets(nx, ny, rl, rv, 200.0, [(nx / 4, ny / 2), (3 * nx / 4, ny / 2)])
    _, info = same(cfg, rho0, (8,))
    assert info["steps_per_launch"] > 1


def test_periodic():
    cfg = p_cfg(1450, 1400, a=0.25, Tr=0.75, **P_KW)
    rng = np.random.default_rng(2)
    rho0 = 0.2 * (1 + 0.05 * rng.uniform(-1, 1, size=(cfg.ny, cfg.nx)))
    same(cfg, rho0, (1, 2, 1, 5))
