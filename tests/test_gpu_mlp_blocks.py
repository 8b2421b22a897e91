"""The surrogate's matrix-core kernels at their edges: tiles of 16 samples with
remainders, workgroups that walk several tiles (more than 128 of them in the
gradient, more than 512 in the forward pass), parameters that are not 16-byte
aligned, and the training step against its two halves.  All comparisons are
between calls of the library whose arithmetic is the same, so they are exact.
"""
import numpy as np
import pytest

from paper_2403_11167_amd import lbm
from test_gpu_mlp import dev, setup, t32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
def test_forward_of_a_sample_does_not_depend_on_its_tile(bf16):
    import torch
    n = 16 * 513 + 5  # one workgroup walks two tiles, the last one partly filled
    x, _, theta, norm = setup(n, seed=21)
    p, xt = t32(theta), t32(x)
    y = lbm.mlp_forward(p, norm, xt, bf16=bf16)
    for a, b in ((0, 1), (3, 18), (16 * 512 - 7, n), (n - 1, n)):
        assert torch.equal(y[a:b], lbm.mlp_forward(p, norm, xt[a:b].contiguous(), bf16=bf16))
    assert torch.isfinite(y).all()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_parameters_need_no_alignment(shift, bf16):
    import torch
    x, y, theta, norm = setup(50, seed=22)
    buf = torch.empty(lbm.MLP_NPARAMS + 4, dtype=torch.float32, device=dev())
    q = buf[shift:shift + lbm.MLP_NPARAMS]
    p = t32(theta)
    q.copy_(p)
    assert q.data_ptr() % 16 == 4 * shift
    assert torch.equal(lbm.mlp_forward(p, norm, t32(x), bf16=bf16),
                       lbm.mlp_forward(q, norm, t32(x), bf16=bf16))
    a = lbm.mlp_grad(p, norm, t32(x), t32(y), bf16=bf16)
    b = lbm.mlp_grad(q, norm, t32(x), t32(y), bf16=bf16)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n", [1, 15, 17, 2048, 2049])
def test_training_step_is_gradient_then_adam(n, bf16):
    import torch
    x, y, theta, norm = setup(n, seed=23)
    s = lbm.Surrogate(theta, bf16=bf16)
    s.norm = norm
    rng = np.random.default_rng(1)
    s.fit(x, y, epochs=1, batch=n, lr=1e-3, seed=1)
    idx = torch.from_numpy(rng.permutation(n).astype(np.int32)).to(dev())
    p, m, v = t32(theta), t32(np.zeros_like(theta)), t32(np.zeros_like(theta))
    _, g = lbm.mlp_grad(p, norm, t32(x), t32(y), idx=idx, bf16=bf16)
    lbm.mlp_adam(p, m, v, g, 1, 1e-3)
    assert torch.isfinite(g).all() and float(g.abs().max()) > 0
    for a, b in ((s.params, p), (s.m, m), (s.v, v)):
        assert torch.equal(a, b)
