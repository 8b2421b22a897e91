"""Patch launches (several steps of a small lattice per launch, in LDS).

Every node does the single-step kernels' arithmetic in the same order, so a
lattice on the default launch shape must equal the same lattice on explicit
strips bit for bit: tiles with remainders in both directions, dimensions that
one tile spans (wrapped inside LDS, down to a single row or column), step
counts that leave a shorter last launch, walls, gravity and the collision
drive with its switch-on inside a launch, and the clamp flag.
"""
import dataclasses

import numpy as np
import pytest

from oracle import theory as th
from paper_2403_11167_amd import inputs, lbm
from test_gpu_parity import fe_cfg, p_cfg, torch_dev
from test_gpu_two_step import FE_TAU, noisy

pytestmark = pytest.mark.gpu

STRIPS = lbm.KF_SET | lbm.KF_NT_STORE
P_KW = dict(tau=[1.0, 0.8, 1.3, 1.0, 0.7, 1.0, 0.7, 1.1, 1.1], sigma_li=0.12, kappa_p=0.7,
            kappa_li=0.3)


def run(cfg, rho0, chunks):
    import torch
    sim = lbm.Simulation(cfg, torch.from_numpy(np.ascontiguousarray(rho0)).to(torch_dev()))
    info = sim.launch_info()
    for n in chunks:
        sim.step(n)
    obs, fields = sim.observe(fields=True)
    f = sim.populations()
    sim.close()
    return obs, [v.cpu().numpy() for v in fields], f.cpu().numpy(), info


def same(cfg, rho0, chunks, walls=False):
    o1, v1, f1, _ = run(cfg.with_launch(64 if cfg.nx < 256 else 256, 0, STRIPS), rho0, chunks)
    o2, v2, f2, info = run(cfg, rho0, chunks)
    assert info["workgroups"] > 0  # the patch path: its shape is fixed before the first step
    assert o1["flags"] == o2["flags"]
    for a, b in zip(v1, v2):
        assert np.array_equal(a, b), float(np.abs(a - b).max())
    if not walls:  # a checkpoint's entries that enter a wall row are unspecified
        assert np.array_equal(f1, f2)
    return o2, info


SIZES = [(1, 1), (1, 40), (40, 1), (2, 3), (5, 7), (33, 20), (64, 8), (70, 66), (257, 9), (101, 50),
         (130, 128), (300, 130), (513, 310), (1000, 777)]


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("model", ["P", "FE"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_patch_equals_strips(nx, ny, model, prec):
    cfg = (p_cfg(nx, ny, a=0.25, Tr=0.75, precision=prec, **P_KW) if model == "P"
           else fe_cfg(nx, ny, a=0.25, Tr=0.75, tau=FE_TAU, precision=prec))
    o, _ = same(cfg, noisy(cfg), (1, 2, 20))
    assert o["flags"] == 0 and o["step"] == 23


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("model", ["P", "FE"])
@pytest.mark.parametrize("nx,ny", [(1, 3), (5, 4), (40, 3), (101, 50), (66, 129), (400, 300)])
def test_patch_walls_equal_strips(nx, ny, model, prec):
    """Channels with a tangential and a normal force; free energy with
    gravity too."""
    kw = dict(walls=True, fx=1e-6, fy=-2e-6, precision=prec)
    cfg = (p_cfg(nx, ny, a=0.25, Tr=0.8, **P_KW, **kw) if model == "P"
           else fe_cfg(nx, ny, a=0.25, Tr=0.8, tau=FE_TAU, g=1e-6, grav_rho0=0.2,
                       grav_y0=0.5 * (ny - 1), **kw))
    rl, rv, _ = th.maxwell(cfg.eos, cfg.a, cfg.b, cfg.R, cfg.T)
    rho0 = inputs.layered(nx, ny, rl, rv, y_i=0.4 * ny)
    rho0 *= 1 + 0.01 * np.random.default_rng(5).uniform(-1, 1, size=rho0.shape)
    same(cfg, rho0, (3, 19), walls=True)


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("model", ["P", "FE"])
@pytest.mark.parametrize("nx,ny", [(200, 100), (131, 45)])
def test_patch_drive_equals_strips(nx, ny, model, prec):
    """The drive switches on at step 10, inside what would be one launch."""
    base = p_cfg(nx, ny, a=0.25, Tr=0.8) if model == "P" else fe_cfg(nx, ny, a=0.25, Tr=0.8)
    cfg = dataclasses.replace(base, ax=5e-4, x_split=nx // 2, ax_from_step=10, precision=prec)
    rl, rv, _ = th.maxwell(cfg.eos, cfg.a, cfg.b, cfg.R, cfg.T)
    rho0 = inputs.droplets(nx, ny, rl, rv, 15.0, [(nx / 4, ny / 2), (3 * nx / 4, ny / 2)])
    same(cfg, rho0, (24,))


def test_patch_clamp_flag():
    a, b, R, T = 9 / 49, 2 / 21, 1.0, 0.8 * 4 / 7
    rl, rv, _ = th.maxwell(th.VDW, a, b, R, T)
    rho0 = inputs.planar_slab(256, 4, rl, rv, width=5.0, noise=1e-6, seed=1)
    cfg = lbm.Config(256, 4, lbm.MODEL_P, lbm.EOS_VDW, a, b, R, T)
    o, info = same(cfg, rho0, (200,))
    assert o["flags"] == lbm.FLAG_PSI_CLAMP and info["steps_per_launch"] > 2
