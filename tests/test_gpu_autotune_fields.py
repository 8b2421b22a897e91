"""The launch fields that the autotuner returns for a lattice on patches: the
patch flag beside the fastest strip shape it timed, which a batch too large
for patches then runs."""
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_batch_patch_classes import config, starts

pytestmark = pytest.mark.gpu
CHOSEN = lbm.KF_REGCAP | lbm.KF_PIPELINE | lbm.KF_TWO_STEP


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("model", [lbm.MODEL_P, lbm.MODEL_FE])
def test_patch_flag_comes_with_the_fastest_strips(model, prec):
    import torch
    cfg = config(512, 512, model, prec)
    r0 = starts([cfg])[0]
    q, ms = lbm.autotune(cfg, r0, steps=10)
    kf = q.kernel_flags & 0xFFFFFFFF
    assert kf & lbm.KF_SET and kf & lbm.KF_PATCH and 0 < ms
    assert q.tile_x in (64, 256) and q.tile_y in (0, 8, 16, 32, 64)
    # plain row loops without any of these are 1.3 times slower or more here
    assert kf & CHOSEN
    sim = lbm.Simulation(q, r0)
    assert sim.launch_info()["workgroups"] > 0  # patches
    sim.close()
    n = 20  # 5.2 M nodes: strips
    b = lbm.Batch([q] * n, [r0] * n)
    b.run(check_every=4, du_tol=0.0, max_steps=8)
    i = b.launch_info(0)
    b.close()
    torch.cuda.synchronize()
    assert i["segment"] == q.tile_y or q.tile_y == 0
    assert i["steps_per_launch"] == (2 if kf & lbm.KF_TWO_STEP and q.tile_x == 256 else 1)
