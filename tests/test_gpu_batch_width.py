"""Strip widths of batch lattices of 128 to 255 columns whose launch shape is
left to the library, in batches too large for patches: partly filled
256-column strips (two steps per launch) only where they are the faster ones,
with the results of whole 64-column strips."""
import numpy as np
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_batch_patch_classes import config, run, same, starts

pytestmark = pytest.mark.gpu
P, FE, F64, F32 = lbm.MODEL_P, lbm.MODEL_FE, lbm.FP64, lbm.FP32_SHIFTED


@pytest.mark.parametrize("model,prec,nx,wide", [
    (P, F64, 128, False), (P, F64, 160, False), (P, F64, 223, False), (P, F64, 224, True),
    (FE, F64, 128, True), (FE, F64, 129, False), (FE, F64, 223, False), (FE, F64, 224, True),
    (P, F32, 127, False), (P, F32, 128, True), (P, F32, 255, True),
    (FE, F32, 128, True), (FE, F32, 129, False), (FE, F32, 175, False), (FE, F32, 176, True)])
def test_width(model, prec, nx, wide):
    ny = 3600000 // (2 * nx)
    cfgs = [config(nx, ny, model, prec) for _ in range(2)]
    r0s = starts(cfgs)
    a = run(cfgs, r0s, [(6, 12, None)])
    b = run([c.with_launch(64, 0, 0) for c in cfgs], r0s, [(6, 12, None)])
    same(a, b)
    for i in a[2][0]:
        assert i["steps_per_launch"] == (2 if wide else 1)
        assert i["threads"] == (64 if not wide else 320 if model == P else 192)
