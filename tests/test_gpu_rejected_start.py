"""A start that is rejected because of its initial density leaves the workspace
as it was: every byte of it, and a lattice or batch that is running there."""
import ctypes

import numpy as np
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_parity import p_cfg
from test_gpu_rho0_check import dev
from test_gpu_two_step import noisy

pytestmark = pytest.mark.gpu


def start(cfg, workspace, rho0):
    import torch
    p, out = cfg.c_params(), ctypes.c_void_p()
    return lbm.lib().lbm_init(ctypes.byref(p), ctypes.c_void_p(workspace.data_ptr()),
                              workspace.numel(), ctypes.c_void_p(rho0.data_ptr()),
                              ctypes.c_void_p(torch.cuda.current_stream().cuda_stream),
                              ctypes.byref(out))


def bad(cfg):
    r = np.full((cfg.ny, cfg.nx), 0.1)
    r[-1, -1] = np.nan
    return dev(r)


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("nx,ny", [(7, 5), (16385, 1), (300, 130), (2100, 1100)])
def test_workspace_bytes(nx, ny, prec):
    import torch
    cfg = p_cfg(nx, ny, a=0.25, Tr=0.75, precision=prec)
    ws = torch.randint(0, 256, (lbm.workspace_bytes(cfg),), dtype=torch.uint8, device="cuda:0")
    was = ws.clone()
    assert start(cfg, ws, bad(cfg)) == lbm.ERR_EOS_DOMAIN
    assert torch.equal(ws, was)
    p, best, ms = cfg.c_params(), lbm.Params(), ctypes.c_double()
    st = lbm.lib().lbm_autotune(ctypes.byref(p), ctypes.c_void_p(ws.data_ptr()), ws.numel(),
                                ctypes.c_void_p(bad(cfg).data_ptr()), None, 1, ctypes.byref(best),
                                ctypes.byref(ms))
    assert st == lbm.ERR_EOS_DOMAIN
    assert torch.equal(ws, was)


@pytest.mark.parametrize("other", [False, True])
def test_running_lattice(other):
    """A start on the workspace of a running lattice, with its own shape or
    another one, is rejected; the lattice goes on."""
    import torch
    cfg = p_cfg(300, 130, a=0.25, Tr=0.75)
    new = p_cfg(150, 130, a=0.25, Tr=0.75) if other else cfg
    rho0 = dev(noisy(cfg))
    a, b = lbm.Simulation(cfg, rho0), lbm.Simulation(cfg, rho0)
    for sim in (a, b):
        sim.step(5)
        sim.observe()
    assert start(new, a.workspace, bad(new)) == lbm.ERR_EOS_DOMAIN
    for sim in (a, b):
        sim.step(5)
    assert a.observe()["du_max"] == b.observe()["du_max"]
    assert torch.equal(a.populations(), b.populations())
    a.close()
    b.close()


def test_running_batch():
    import torch
    cfgs = [p_cfg(300, 130, a=0.25, Tr=0.75), p_cfg(150, 130, a=0.25, Tr=0.75)]
    r0s = [dev(noisy(c)) for c in cfgs]
    a, b = lbm.Batch(cfgs, r0s), lbm.Batch(cfgs, r0s)
    for x in (a, b):
        x.run(check_every=4, du_tol=0.0, max_steps=8)
    p = (lbm.Params * 2)(*[c.c_params() for c in cfgs])
    broken = bad(cfgs[1])
    ptrs = (ctypes.c_void_p * 2)(r0s[0].data_ptr(), broken.data_ptr())
    out = ctypes.c_void_p()
    was = a.workspace.clone()
    st = lbm.lib().lbm_batch_create(2, p, ptrs, ctypes.c_void_p(a.workspace.data_ptr()),
                                    a.workspace.numel(),
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream),
                                    ctypes.byref(out))
    assert st == lbm.ERR_EOS_DOMAIN and torch.equal(a.workspace, was)
    for x in (a, b):
        for i in range(2):
            x.set_limit(i, 1 << 40)
        x.run(check_every=4, du_tol=0.0, max_steps=8)
    assert a.state() == b.state()
    for i in range(2):
        for u, v in zip(a.observe(i, fields=True)[1], b.observe(i, fields=True)[1]):
            assert torch.equal(u, v)
    a.close()
    b.close()
