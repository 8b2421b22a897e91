"""Patches at the sizes where they hold two nodes per thread and take several
rounds of workgroups: channels with gravity, the collision drive and periodic
lattices, up to 3 M nodes, against the same lattice on explicit strips, bit
for bit (every node does the same arithmetic in the same order)."""
import dataclasses

import numpy as np
import pytest

from oracle import theory as th
from paper_2403_11167_amd import inputs, lbm
from test_gpu_parity import fe_cfg, p_cfg
from test_gpu_patch import P_KW, same
from test_gpu_two_step import FE_TAU, noisy

pytestmark = pytest.mark.gpu


def nodes_per_thread(cfg, info):
    """1 or 2, from the cells a workgroup holds (tile and halo; a spanned
    dimension has no halo, but then the whole lattice's cells)."""
    halo = (2 if cfg.model == lbm.MODEL_P else 3) * info["steps_per_launch"] - 1
    w = info["strip"] + (2 if info["strip"] == cfg.nx else 2 * halo)
    h = info["segment"] + (0 if info["segment"] == cfg.ny and not cfg.walls else 2 * halo)
    return -(-w * h // info["threads"])


def channel(nx, ny, model, prec):
    kw = dict(walls=True, fx=1e-6, fy=-2e-6, precision=prec)
    cfg = (p_cfg(nx, ny, a=0.25, Tr=0.8, **P_KW, **kw) if model == "P"
           else fe_cfg(nx, ny, a=0.25, Tr=0.8, tau=FE_TAU, g=1e-6, grav_rho0=0.2,
                       grav_y0=0.5 * (ny - 1), **kw))
    rl, rv, _ = th.maxwell(cfg.eos, cfg.a, cfg.b, cfg.R, cfg.T)
    rho0 = inputs.layered(nx, ny, rl, rv, y_i=0.4 * ny)
    return cfg, rho0 * (1 + 0.01 * np.random.default_rng(5).uniform(-1, 1, size=rho0.shape))


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("model", ["P", "FE"])
@pytest.mark.parametrize("nx,ny", [(512, 513), (701, 500), (1030, 1021)])
def test_wide_channels_equal_strips(nx, ny, model, prec):
    cfg, rho0 = channel(nx, ny, model, prec)
    _, info = same(cfg, rho0, (1, 2, 13), walls=True)
    if not (model == "FE" and prec == lbm.FP64):  # that kernel exists with one node per thread
        assert nodes_per_thread(cfg, info) == 2


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("model", ["P", "FE"])
def test_drive_on_a_wide_lattice_equals_strips(model, prec):
    """The drive switches on at step 7, inside what would be one launch."""
    nx, ny = 1000, 600
    base = p_cfg(nx, ny, a=0.25, Tr=0.8) if model == "P" else fe_cfg(nx, ny, a=0.25, Tr=0.8)
    cfg = dataclasses.replace(base, ax=5e-4, x_split=nx // 2, ax_from_step=7, precision=prec)
    rl, rv, _ = th.maxwell(cfg.eos, cfg.a, cfg.b, cfg.R, cfg.T)
    rho0 = inputs.droplets(nx, ny, rl, rv, 100.0, [(nx / 4, ny / 2), (3 * nx / 4, ny / 2)])
    _, info = same(cfg, rho0, (17,))
    if not (model == "FE" and prec == lbm.FP64):
        assert nodes_per_thread(cfg, info) == 2


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
def test_several_rounds_of_the_general_form(prec):
    """3 M nodes of a channel, P: several rounds of workgroups (FE leaves the
    patches at 1.8 M nodes)."""
    cfg, rho0 = channel(1999, 1501, "P", prec)
    _, info = same(cfg, rho0, (2, 9), walls=True)
    assert info["workgroups"] > 1024 and nodes_per_thread(cfg, info) == 2


@pytest.mark.parametrize("model,nx,ny,prec", [("P", 1400, 1301, lbm.FP64),
                                              ("P", 1400, 1301, lbm.FP32_SHIFTED),
                                              ("FE", 901, 900, lbm.FP64),
                                              ("FE", 1201, 1101, lbm.FP32_SHIFTED)])
def test_several_rounds_of_the_periodic_form(model, nx, ny, prec):
    cfg = (p_cfg(nx, ny, a=0.25, Tr=0.75, precision=prec, **P_KW) if model == "P"
           else fe_cfg(nx, ny, a=0.25, Tr=0.75, tau=FE_TAU, precision=prec))
    same(cfg, noisy(cfg), (1, 2, 10))
