"""The launch shape that a batch reports of a lattice that has retired is the
one it last ran with, whatever its family runs with now."""
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_batch_patch_classes import config, on_patches, starts

pytestmark = pytest.mark.gpu


def go_on(b, which):
    for i in which:
        b.set_limit(i, 1 << 40)
    b.run(check_every=4, du_tol=0.0, max_steps=8)
    return [b.launch_info(i) for i in range(b.n)]


def test_retired_lattices():
    P, FE, prec = lbm.MODEL_P, lbm.MODEL_FE, lbm.FP32_SHIFTED
    cfgs = [config(64, 64, P, prec), config(300, 200, P, prec), config(70, 45, FE, prec)]
    cfgs += [config(512, 512, P, prec) for _ in range(14)]
    b = lbm.Batch(cfgs, starts(cfgs))
    everyone = go_on(b, range(b.n))
    both = go_on(b, [0, 1])     # the family of P on patches
    assert on_patches(both[0]) and on_patches(both[1]) and both[2] == everyone[2]
    one = go_on(b, [0])         # patches of another shape: lattice 1 keeps its own
    assert on_patches(one[0]) and one[1] == both[1]
    fe = go_on(b, [2])          # no active lattice of P
    assert fe[0] == one[0] and fe[1] == both[1] and on_patches(fe[2])
    for info in (both, one, fe):
        for i in range(3):
            assert info[i]["threads"] >= 64
    b.close()
