"""The observation at the widths where its tiles change (8 x 64, 16 x 32, 32 x
16 or 64 x 8 nodes; up to 512 tiles always 64 x 8): several tiles with
remainders in both directions, periodic and between walls, against the oracle,
and several rounds of tiles against the sums of the exported fields."""
import math

import numpy as np
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_observe import test_observe_matches_oracle as matches_oracle
from test_gpu_parity import fe_cfg, p_cfg
from test_gpu_two_step import noisy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", ["P", "FE"])
@pytest.mark.parametrize("nx,ny,walls", [(1, 4096, False), (1, 4097, False), (3, 4500, False),
                                         (8, 4161, False), (9, 4099, False), (16, 4129, False),
                                         (17, 4111, False), (32, 4112, False), (33, 4113, False),
                                         (65, 2064, False), (96, 2065, False), (97, 2065, False),
                                         (288, 830, False), (1, 4161, True), (9, 4160, True),
                                         (16, 4130, True), (32, 4130, True), (33, 4130, True),
                                         (65, 2070, True)])
def test_widths(nx, ny, walls, model):
    matches_oracle(nx, ny, walls, model)


@pytest.mark.parametrize("model", ["P", "FE"])
def test_more_tiles_than_workgroups(model):
    """5 x 140000: 2188 tiles on 2048 workgroups."""
    import torch
    cfg = p_cfg(5, 140000, a=0.25) if model == "P" else fe_cfg(5, 140000)
    sim = lbm.Simulation(cfg, torch.from_numpy(np.ascontiguousarray(noisy(cfg))).to("cuda:0"))
    sim.step(2)
    o, (rho, ux, uy) = sim.observe(3, 70001, fields=True)
    sim.close()
    r = rho.cpu().numpy()
    u = torch.sqrt(ux * ux + uy * uy).cpu().numpy()
    assert math.isclose(o["mass"], math.fsum(r.ravel()), rel_tol=1e-15)
    assert (o["rho_min"], o["rho_max"]) == (r.min(), r.max())
    assert math.isclose(o["max_u"], u.max(), rel_tol=1e-15)
    assert o["rho_in"] == r[70001, 3] and o["rho_out"] == r[1, 0]
