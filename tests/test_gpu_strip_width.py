"""Strip widths of the two-step kernels on one lattice: the strips are equal,
start on multiples of 16 columns and leave the last 16 lanes of a workgroup
of 128, 192 or 256 lanes to the halo columns.  At the widths where their
number or width changes, two steps must equal two single steps bit for bit
(the arithmetic of a node is the same in the same order)."""
import numpy as np
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_parity import fe_cfg, p_cfg
from test_gpu_two_step import FE_TAU, FE_VARIANTS, ONE, TWO, noisy, run

pytestmark = pytest.mark.gpu

WIDTHS = [1, 15, 17, 112, 113, 176, 177, 225, 240, 241, 353, 480, 481, 1000]


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("nx", WIDTHS)
def test_p_strip_widths(nx, prec):
    cfg = p_cfg(nx, 21, a=0.25, Tr=0.75, tau=[1.0, 0.8, 1.3, 1.0, 0.7, 1.0, 0.7, 1.1, 1.1],
                sigma_li=0.12, kappa_p=0.7, kappa_li=0.3, precision=prec)
    rho0 = noisy(cfg)
    o1, r1, f1 = run(cfg.with_launch(256, 10, ONE), rho0, 8)
    o2, r2, f2 = run(cfg.with_launch(256, 10, TWO), rho0, 8)
    assert o1["flags"] == o2["flags"]
    assert np.array_equal(f1, f2) and np.array_equal(r1, r2)


@pytest.mark.parametrize("variant", list(FE_VARIANTS))
@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("nx", WIDTHS)
def test_fe_strip_widths(nx, prec, variant):
    cfg = fe_cfg(nx, 21, a=0.25, Tr=0.75, tau=FE_TAU, precision=prec)
    rho0 = noisy(cfg)
    o1, r1, f1 = run(cfg.with_launch(256, 10, ONE), rho0, 8)
    o2, r2, f2 = run(cfg.with_launch(256, 10, FE_VARIANTS[variant]), rho0, 8)
    assert o1["flags"] == o2["flags"]
    assert np.array_equal(f1, f2) and np.array_equal(r1, r2)
