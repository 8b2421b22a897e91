"""The two-step FP32 pseudopotential kernel forms its square roots by an
estimate and one residual step, the single-step kernels by sqrtf.  The two
agree for every float of [2^-60, 2^60] only because of what the hardware's
estimate is there, so the kernels are compared at as many arguments as there
are: lattices whose densities are spread over two binades (a root depends on
its argument's mantissa and on whether the exponent is odd), eight times the
2^24 different arguments in each of the two steps, and lattices with arguments
on either side of 2^-60."""
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_two_step import ONE, TWO

pytestmark = pytest.mark.gpu


def populations(cfg, rho0):
    sim = lbm.Simulation(cfg, rho0)
    sim.step(2)
    flags = sim.observe()["flags"]
    f = sim.populations()
    sim.close()
    return flags, f


def same(nx, ny, rho0, T):
    import torch
    # psi^2 = 2 rho (1/3 - R T / (1 - b rho)) with a = 0
    cfg = lbm.Config(nx, ny, lbm.MODEL_P, lbm.EOS_VDW, 0.0, 1e-3, 1.0, T,
                     precision=lbm.FP32_SHIFTED)
    a = populations(cfg.with_launch(256, 64, ONE), rho0)
    b = populations(cfg.with_launch(256, 64, TWO), rho0)
    assert a[0] == b[0]
    assert torch.equal(torch.nan_to_num(a[1]), torch.nan_to_num(b[1]))
    assert torch.equal(torch.isnan(a[1]), torch.isnan(b[1]))


@pytest.mark.parametrize("seed", range(8))
def test_every_argument(seed):
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    n = 4096
    u = torch.rand((n, n), generator=g, device="cuda:0", dtype=torch.float64)
    same(n, n, 1.0 + 3.0 * u, 1e-2 * (1 + seed))


def test_either_side_of_the_range():
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(99)
    u = torch.rand((512, 512), generator=g, device="cuda:0", dtype=torch.float64)
    same(512, 512, torch.exp2(-66.0 + 10.0 * u), 1e-2)
