"""The one-pass observation at the edges of its 64 x 8 tiles, against the
oracle: remainders in both directions, lattices narrower than a stencil halo,
channels of three and more rows, and a lattice of more tiles than workgroups
(against the sums of its own exported fields)."""
import math

import numpy as np
import pytest

from oracle import theory as th
from paper_2403_11167_amd import inputs, lbm
from test_gpu_parity import FP64_RTOL, fe_cfg, oracle_run, p_cfg, rel_err, torch_dev
from test_gpu_two_step import noisy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", ["P", "FE"])
@pytest.mark.parametrize("nx,ny,walls", [(1, 1, False), (2, 3, False), (63, 7, False),
                                         (64, 8, False), (65, 9, False), (129, 17, False),
                                         (5, 3, True), (64, 8, True), (70, 25, True)])
def test_observe_matches_oracle(nx, ny, walls, model):
    import torch
    kw = dict(walls=True, fx=1e-6) if walls else {}
    cfg = (p_cfg(nx, ny, a=0.25, **kw) if model == "P" else fe_cfg(nx, ny, **kw))
    if walls:
        rl, rv, _ = th.maxwell(cfg.eos, cfg.a, cfg.b, cfg.R, cfg.T)
        rho0 = inputs.layered(nx, ny, rl, rv)
    else:
        rho0 = noisy(cfg)
    sim = lbm.Simulation(cfg, torch.from_numpy(np.ascontiguousarray(rho0)).to(torch_dev()))
    ref = oracle_run(cfg, rho0, 5)
    sim.step(5)
    first, (rho, ux, uy) = sim.observe(nx // 2, ny // 2, fields=True)
    again = sim.observe(nx // 2, ny // 2)
    sim.close()
    rr, uxr, uyr = ref.fields()
    o = ref.observe(nx // 2, ny // 2)
    assert rel_err(rho.cpu().numpy(), rr) < FP64_RTOL
    umax = max(float(np.abs(uxr).max()), float(np.abs(uyr).max()), 1e-12)
    for a, b in ((ux, uxr), (uy, uyr)):
        assert np.max(np.abs(a.cpu().numpy() - b)) < 1e-8 * max(umax, 1e-6)
    r = rho.cpu().numpy()
    assert math.isclose(first["mass"], math.fsum(r.ravel()), rel_tol=1e-15)
    assert (first["rho_min"], first["rho_max"]) == (r.min(), r.max())
    assert math.isclose(first["rho_in"], o["rho_in"], rel_tol=1e-10)
    assert math.isclose(first["rho_out"], o["rho_out"], rel_tol=1e-10)
    assert first["flags"] == ref.flags
    # the state has not moved: the second call, without exports, agrees and
    # measures no change of velocity
    assert math.isinf(first["du_max"]) and again["du_max"] == 0.0
    for k in ("mass", "max_u", "rho_min", "rho_max", "dp"):
        assert first[k] == again[k] or (math.isnan(first[k]) and math.isnan(again[k]))


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
def test_observe_walks_several_tiles(prec):
    """1500 x 1100: 3312 tiles on 2048 workgroups."""
    import torch
    cfg = fe_cfg(1500, 1100, precision=prec)
    rho0 = noisy(cfg)
    sim = lbm.Simulation(cfg, torch.from_numpy(np.ascontiguousarray(rho0)).to(torch_dev()))
    sim.step(2)
    o, (rho, ux, uy) = sim.observe(700, 500, fields=True)
    sim.close()
    r = rho.cpu().numpy()
    u = torch.sqrt(ux * ux + uy * uy).cpu().numpy()
    assert math.isclose(o["mass"], math.fsum(r.ravel()), rel_tol=1e-15)
    assert (o["rho_min"], o["rho_max"]) == (r.min(), r.max())
    assert math.isclose(o["max_u"], u.max(), rel_tol=1e-15)
    assert o["rho_in"] == r[500, 700] and o["rho_out"] == r[(500 + 550) % 1100, (700 + 750) % 1500]
