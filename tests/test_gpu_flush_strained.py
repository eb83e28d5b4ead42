"""The flush of patches of loose triangles with two unknowns per vertex, FP32, on strongly stretched elements, whose
gradients do not cancel: every entry against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from . import parity as PR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [1 | 2 | 4, 1 | 2 | 4 | 8])
@pytest.mark.parametrize("k", [170, 171, 172, 342, 512])      # 3 k vertices, 6 k blocks of the upper half
def test_loose_stretched_triangles(k, mode):
    import torch
    print("[case] flush, stretched", k, mode, flush=True)
    r = np.random.default_rng(20 * k)
    one = np.array([[0.0, 0.0, 0.0], [1.0, 0.0, 0.0], [0.2, 0.9, 0.0]])
    rest = (one[None] + 0.1 * r.normal(size=(k, 3, 3)) * [1, 1, 0]).reshape(-1, 3)
    tris = np.arange(3 * k, dtype=np.int32).reshape(k, 3)
    x = (rest.reshape(k, 3, 3)[:, :, :2] @ np.array([[1.8, 0.3], [0.0, 1.4]]) + 0.05 * r.normal(size=(k, 3, 2))).reshape(-1, 2)
    _, prob = PR.build_gpu(tris, rest, 3 * k, 2, [(6, ())], 1, patch_faces=512)
    P = PR.build_oracle(tris, rest, 3 * k, 2, [(6, ())])
    ref = P.eval(x.ravel(), mode)
    e, g, h = (t.cpu().numpy() for t in prob.eval(torch.from_numpy(x.ravel()).cuda(), mode))
    rtol = PR.RTOL[1]
    assert abs(e[0] - ref.energy) <= rtol * ref.esum_abs
    PR.assert_close("grad", g, ref.grad, ref.gscale, rtol)
    PR.assert_close("hess", h, ref.hess, ref.hscale, rtol)
