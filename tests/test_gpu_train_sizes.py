"""Training gradient at the sizes where its work is split: part of a workgroup, one, several, and more samples than
one round of all workgroups, against reverse-mode FP64 (PyTorch on the CPU)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2509_00406_amd import mad

from .test_gpu_mlp import oracle_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 3, 4, 5, 127, 2048, 2049, 4100])
@pytest.mark.parametrize("indexed", [False, True])
def test_loss_gradient(count, indexed):
    import torch
    print("training gradient", count, indexed, flush=True)
    r = np.random.default_rng(count)
    n, base = count + 37, 11
    z = (r.normal(size=(n, 6)) * (1e-2, 1e-2, 1e-2, 0.3, 0.3, 0.3)).astype(np.float32)
    W, dW = r.normal(size=n).astype(np.float32), r.normal(size=(n, 6)).astype(np.float32)
    th = np.concatenate([r.normal(0, 0.5, 448), r.normal(0, 0.125, 4096), r.normal(0, 0.5, 64),
                         r.normal(0, 0.0625, 64), [0.1]]).astype(np.float32)
    s_in, c_g = np.array([30, 30, 30, 3, 3, 3], np.float32), np.full(6, 0.7, np.float32)
    idx = r.permutation(n).astype(np.int32)
    net = mad.Network(th, s_in, 0.5)
    t = [torch.from_numpy(a).cuda() for a in (z, W, dW)]
    g, loss = net.loss_grad(*t, 1.3, c_g, 0.8, idx=torch.from_numpy(idx).cuda() if indexed else None, base=base,
                            count=count)
    at = idx[base:base + count] if indexed else np.arange(base, base + count)
    loss_ref, g_ref = O.mlp_loss_grad(oracle_params(th, s_in, 0.5), z[at], W[at], dW[at], 1.3, c_g, 0.8)
    # the tolerance of the training gradient in test_gpu_mlp.py: relative to the largest entry
    assert np.abs(g.cpu().numpy() - g_ref).max() <= 5e-6 * np.abs(g_ref).max()
    assert abs(float(loss) - loss_ref) <= 5e-6 * abs(loss_ref)
    g2, _ = net.loss_grad(*t, 1.3, c_g, 0.8, idx=torch.from_numpy(idx).cuda() if indexed else None, base=base, count=count)
    assert torch.equal(g, g2)   # fixed order of the sums
