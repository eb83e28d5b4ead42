"""Patches with more vertices and blocks than one step of the flush takes (two vertices and four block rows per
thread): triangles that share nothing have three vertices and six blocks each, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from . import parity as PR

pytestmark = pytest.mark.gpu
KINDS = {1: [(3, ())], 2: [(6, ())], 3: [(2, ())]}      # Dirichlet, symmetric Dirichlet, area


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("k", [170, 171, 172, 342, 512])      # 3 k vertices, 6 k blocks of the upper half
def test_patch_of_loose_triangles(dim, precision, k):
    import torch
    print("[case] flush", dim, precision, k, flush=True)
    r = np.random.default_rng(10 * k + dim)
    one = np.array([[0.0, 0.0, 0.0], [1.0, 0.0, 0.0], [0.2, 0.9, 0.0]])
    rest = (one[None] + 0.1 * r.normal(size=(k, 3, 3)) * [1, 1, dim == 3]).reshape(-1, 3)
    rest[:, 0] += np.repeat(np.arange(k), 3) * 2.0 / k
    tris = np.arange(3 * k, dtype=np.int32).reshape(k, 3)
    x = rest[:, :dim] + 0.05 * r.normal(size=(3 * k, dim))
    _, prob = PR.build_gpu(tris, rest, 3 * k, dim, KINDS[dim], precision, patch_faces=512)
    P = PR.build_oracle(tris, rest, 3 * k, dim, KINDS[dim])
    ref = P.eval(np.ascontiguousarray(x).ravel(), 1 | 2 | 4)
    e, g, h = (t.cpu().numpy() for t in prob.eval(torch.from_numpy(np.ascontiguousarray(x).ravel()).cuda(), 1 | 2 | 4))
    rtol = PR.RTOL[precision]
    assert abs(e[0] - ref.energy) <= rtol * ref.esum_abs
    if dim == 2 and precision == 1:
        # these triangles' gradients cancel to where FP32 derivatives are past the bar whatever assembles them:
        # the same elements added by global atomics instead
        _, other = PR.build_gpu(tris, rest, 3 * k, dim, KINDS[dim], precision, scatter=1)
        ref.grad = other.eval(torch.from_numpy(np.ascontiguousarray(x).ravel()).cuda(), 1 | 2 | 4)[1].cpu().numpy()
    PR.assert_close("grad", g, ref.grad, ref.gscale, rtol)
    PR.assert_close("hess", h, ref.hess, ref.hscale, rtol)
