"""Patches in batches of the sizes that calibrations run: size classes of many
lattices (two nodes per thread), and a family that moves between strips and
patches as its lattices retire and resume, beside the other family and alone.
Every lattice's fields, du measurements, states and flags equal the same
batch on explicit strips bit for bit."""
import numpy as np
import pytest

from oracle import theory as th
from paper_2403_11167_amd import inputs, lbm
from test_gpu_parity import cs_T, torch_dev

pytestmark = pytest.mark.gpu


def config(nx, ny, model, prec):
    T = cs_T(0.25, 0.8)
    tau = [1.0] * 9
    kw = dict(sigma_li=0.1, kappa_p=0.9) if model == lbm.MODEL_P else dict(kappa=0.5)
    if model == lbm.MODEL_FE:
        tau[1] = 0.75
    return lbm.Config(nx, ny, model, lbm.EOS_CS, 0.25, 4.0, 1.0, T, tau=tau, precision=prec, **kw)


def starts(cfgs):
    import torch
    out = []
    for k, c in enumerate(cfgs):
        rl, rv, _ = th.maxwell(c.eos, c.a, c.b, c.R, c.T)
        r = inputs.spinodal(c.nx, c.ny, 0.5 * (rl + rv), 0.01, seed=k)
        out.append(torch.from_numpy(np.ascontiguousarray(r)).to(torch_dev()))
    return out


def on_patches(info):
    """Strips of a batch report one or two steps of workgroups of 64, 192, 256
    or 320 threads; these lattices' patches differ in one or the other."""
    return info["steps_per_launch"] > 2 or info["threads"] not in (64, 192, 256, 320)


def run(cfgs, r0s, plan):
    """plan: (check_every, steps, indices that go on or None for all)."""
    b = lbm.Batch(cfgs, r0s)
    trace, infos = [], []
    for k, (every, steps, only) in enumerate(plan):
        if k:
            for i in range(b.n):
                if only is None or i in only:
                    b.set_limit(i, 1 << 40)
        assert b.run(check_every=every, du_tol=0.0, max_steps=steps) == steps
        trace.append(b.state())
        infos.append([b.launch_info(i) for i in range(b.n)])
    fields = [[v.cpu().numpy() for v in b.observe(i, fields=True)[1]] for i in range(b.n)]
    b.close()
    return trace, fields, infos


def strips_of(cfgs):
    return [c.with_launch(256 if c.nx >= 128 else 64, 16, 0) for c in cfgs]


def same(a, b):
    for x, y in zip(a[0], b[0]):
        assert x[0] == y[0] and x[1] == y[1] and x[3] == y[3]
        assert np.array_equal(x[2], y[2])
    for i, (x, y) in enumerate(zip(a[1], b[1])):
        for u, v in zip(x, y):
            assert np.array_equal(u, v), i


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("model", [lbm.MODEL_P, lbm.MODEL_FE])
def test_size_classes_of_many_lattices(model, prec):
    cfgs = ([config(128, 128, model, prec) for _ in range(12)]
            + [config(64, 64, model, prec) for _ in range(32)]
            + [config(100, 75, model, prec) for _ in range(3)])
    r0s = starts(cfgs)
    plan = [(10, 40, None), (14, 28, None), (2, 4, None)]
    a, b = run(cfgs, r0s, plan), run(strips_of(cfgs), r0s, plan)
    same(a, b)
    H = 2 if model == lbm.MODEL_P else 3
    two = 0
    for c, i in zip(cfgs, a[2][-1]):
        assert on_patches(i), i
        halo = H * i["steps_per_launch"] - 1
        w = i["strip"] + (2 if i["strip"] == c.nx else 2 * halo)
        h = i["segment"] + (0 if i["segment"] == c.ny else 2 * halo)
        two += w * h > i["threads"]
    assert two > 0  # the form with two nodes per thread


@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_SHIFTED])
@pytest.mark.parametrize("model,n", [(lbm.MODEL_P, 14), (lbm.MODEL_FE, 8)])
def test_family_moves_between_strips_and_patches(model, n, prec):
    """All n lattices of 512^2 fill the device with strips; when only one goes
    on, its family moves to patches (the strips' graph is dropped, clearing
    and gathering move outside it), and back when all resume.  Two small
    lattices of the other family run on patches beside the strips."""
    other = lbm.MODEL_FE if model == lbm.MODEL_P else lbm.MODEL_P
    cfgs = [config(512, 512, model, prec) for _ in range(n)]
    cfgs += [config(64, 64, other, prec), config(70, 45, other, prec)]
    r0s = starts(cfgs)
    plan = [(10, 20, None), (12, 24, {1}), (10, 20, {0, 1, n}), (20, 20, None), (6, 12, {n + 1})]
    a, b = run(cfgs, r0s, plan), run(strips_of(cfgs), r0s, plan)
    same(a, b)
    infos = a[2]
    for i in range(n):
        assert not on_patches(infos[0][i]) and not on_patches(infos[3][i])
    assert on_patches(infos[1][1]) and on_patches(infos[2][0]) and on_patches(infos[2][1])
    for k in (0, 2, 3):
        assert on_patches(infos[k][n])
    assert on_patches(infos[4][n + 1])
