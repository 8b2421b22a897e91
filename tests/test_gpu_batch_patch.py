"""Batches on patches (the default launch shape of lattices that do not fill
the device): every lattice, its du measurements, states and flags equal the
same batch on explicit strips bit for bit, over check intervals that divide
into full and shortened launches, families of both models and equations of
state with several sizes in one launch, spanned dimensions, resumed runs and
a batch in which only one lattice goes on.
"""
import numpy as np
import pytest

from oracle import theory as th
from paper_2403_11167_amd import inputs, lbm
from test_gpu_parity import cs_T, torch_dev

pytestmark = pytest.mark.gpu


def problems(precision):
    a = 0.25
    T = cs_T(a, 0.8)
    rl, rv, _ = th.maxwell(th.CS, a, 4.0, 1.0, T)
    Tv = 0.9 * 4 / 7
    rlv, rvv, _ = th.maxwell(th.VDW, 9 / 49, 2 / 21, 1.0, Tv)
    tauF = [1.0] * 9
    tauF[1] = 0.75
    P = dict(sigma_li=0.1, kappa_p=0.9, precision=precision)
    F = dict(tau=tauF, kappa=0.5, precision=precision)
    out = []
    for k, (nx, ny) in enumerate([(64, 8), (128, 128), (70, 45), (5, 7), (300, 20)]):
        out.append((lbm.Config(nx, ny, 0, lbm.EOS_CS, a, 4.0, 1.0, T, **P), 0.5 * (rl + rv), k))
        out.append((lbm.Config(nx, ny, 1, lbm.EOS_CS, a, 4.0, 1.0, T, **F), 0.5 * (rl + rv), k + 9))
    out.append((lbm.Config(33, 20, 0, lbm.EOS_VDW, 9 / 49, 2 / 21, 1.0, Tv, precision=precision),
                0.5 * (rlv + rvv), 30))
    return out


def run(cfgs, r0s, plan):
    import torch
    b = lbm.Batch(cfgs, [torch.from_numpy(np.ascontiguousarray(r)).to(torch_dev()) for r in r0s])
    dus = []
    for k, (every, steps, only) in enumerate(plan):
        if k:
            for i in range(b.n):
                if only is None or i == only:
                    b.set_limit(i, 1 << 40)
        assert b.run(check_every=every, du_tol=0.0, max_steps=steps) == steps
        dus.append(b.state()[2])
    info = [b.launch_info(i) for i in range(b.n)]
    st = b.state()
    fields = [[v.cpu().numpy() for v in b.observe(i, fields=True)[1]] for i in range(b.n)]
    stats = b.stats()
    b.close()
    return st, dus, fields, info, stats


@pytest.mark.parametrize("precision", [lbm.FP64, lbm.FP32_SHIFTED])
def test_batch_patches_equal_strips(precision):
    probs = problems(precision)
    r0s = [inputs.spinodal(c.nx, c.ny, m, 0.01, seed=s) for c, m, s in probs]
    auto = [c for c, _, _ in probs]
    strips = [c.with_launch(256 if c.nx >= 128 else 64, 4, 0) for c in auto]
    plan = [(8, 32, None), (10, 30, None), (50, 100, None), (2, 4, None), (38, 76, 3)]
    a, b = run(auto, r0s, plan), run(strips, r0s, plan)
    assert all(i["steps_per_launch"] > 2 for i in a[3][:2])  # on patches
    assert a[0][0] == b[0][0] and a[0][1] == b[0][1] and a[0][3] == b[0][3]
    for x, y in zip(a[1], b[1]):
        assert np.array_equal(x, y)  # du of every lattice after every run
    for i, (x, y) in enumerate(zip(a[2], b[2])):
        for u, v in zip(x, y):
            assert np.array_equal(u, v), i
    assert a[4]["node_updates"] == b[4]["node_updates"]


def test_batch_families_mix_with_strips():
    """A family on patches beside lattices with an explicit strip shape."""
    probs = problems(lbm.FP32_SHIFTED)
    r0s = [inputs.spinodal(c.nx, c.ny, m, 0.01, seed=s) for c, m, s in probs]
    auto = [c for c, _, _ in probs]
    mixed = [c.with_launch(64, 0, 0) if i % 3 == 0 else c for i, c in enumerate(auto)]
    plan = [(20, 60, None), (12, 24, None)]
    a, b = run(auto, r0s, plan), run(mixed, r0s, plan)
    for x, y in zip(a[1], b[1]):
        assert np.array_equal(x, y)
    for x, y in zip(a[2], b[2]):
        for u, v in zip(x, y):
            assert np.array_equal(u, v)
